// Two threads raise the pass kernels' dynamic-LDS limit at once (no GPU).
//
// hipFuncSetAttribute is defined here, ahead of the HIP runtime's, and keeps
// the last value set per kernel.  The thread that asks for less is held inside
// its first call until the other one has finished, or for a while: whatever
// the order, the limit that stands in the end has to be the larger one.
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <map>
#include <mutex>
#include <thread>

#include "sv_pass.h"

static std::mutex mu;
static std::condition_variable cv;
static std::map<const void*, int> attr;
static bool small_inside, large_done;
constexpr int kSmall = 20 << 10, kLarge = 100 << 10;

extern "C" hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int value)
{
    std::unique_lock<std::mutex> lk(mu);
    if (value == kSmall && !small_inside) {
        small_inside = true;
        cv.notify_all();
        cv.wait_for(lk, std::chrono::milliseconds(500), [] { return large_done; });
    }
    attr[f] = value;
    return hipSuccess;
}

int main()
{
    hipError_t ea = hipErrorUnknown, eb = hipErrorUnknown;
    std::thread a([&] { ea = svk::pass_engine_prepare(kSmall); });
    std::thread b([&] {
        {
            std::unique_lock<std::mutex> lk(mu);
            cv.wait(lk, [] { return small_inside; });
        }
        eb = svk::pass_engine_prepare(kLarge);
        std::lock_guard<std::mutex> lk(mu);
        large_done = true;
        cv.notify_all();
    });
    a.join();
    b.join();
    int lowest = 1 << 30;
    for (const auto& kv : attr) lowest = kv.second < lowest ? kv.second : lowest;
    printf("kernels %zu lowest limit %d status %d %d\n", attr.size(), lowest, (int)ea, (int)eb);
    return !attr.empty() && lowest == kLarge && ea == hipSuccess && eb == hipSuccess ? 0 : 1;
}
