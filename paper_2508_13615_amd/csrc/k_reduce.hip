// k_reduce.hip -- measurement reductions for gfx950.
//
// Expectation values of Pauli strings and of Pauli sums (the "measurement
// processes" routines of Sec. 2; Listing 1 takes <H> of a Hamiltonian).
// For P with X/Y positions f = xmask and Z/Y positions zmask:
//   P|x> = i^{nY} (-1)^{popcount(x & zmask)} |x ^ f>,
//   <psi|P|psi> = sum_x conj(psi[x ^ f]) i^{nY} (-1)^{pc(x & zmask)} psi[x].
// For f = 0 this is sum_x |psi_x|^2 (-1)^{pc(x & zmask)}.  For f != 0 the
// terms of x and x ^ f are complex conjugates (P is Hermitian), so only x with
// bit p = 0 (p = top bit of f) is visited and the term counted as 2 Re(.):
// every amplitude is read exactly once.
//
// Accumulation: complex64 loads are widened to fp64 before any product
// (expectations); the norm of a complex64 state sums one chunk per thread
// in fp32 and everything above that in fp64.  Stage 1 writes one fp64
// partial per block of a fixed grid, stage 2 sums partials in fixed order:
// repeated calls give bit-identical results.
#include <algorithm>

#include "sv_core.h"

namespace svk {

// Deterministic block sum (wavefront butterfly, then waves in order).
// Valid on thread 0.
__device__ __forceinline__ double block_sum(double v)
{
    __shared__ double sm[kReduceThreads / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) sm[wave] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0) {
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += sm[w];
    }
    return s;
}

static int reduce_grid(uint64_t n_items)
{
    uint64_t per = (uint64_t)kReduceThreads * 4;
    uint64_t nb = (n_items + per - 1) / per;
    if (nb < 1) nb = 1;
    if (nb > (uint64_t)kReduceBlocks) nb = kReduceBlocks;
    return (int)nb;
}

template <typename T>
__global__ void __launch_bounds__(kReduceThreads)
k_norm_partial(const typename Vec2<T>::type* __restrict__ psi, uint64_t n, double* __restrict__ partials)
{
    using V = typename Vec2<T>::type;
    double acc = 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x * 4;
    for (uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x * 4 + threadIdx.x; i0 < n + threadIdx.x; i0 += stride) {
        V a[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t i = i0 + (uint64_t)j * blockDim.x;
            if (i < n) a[j] = psi[i];
            else { a[j].x = T(0); a[j].y = T(0); }
        }
        T loc = T(0);  // fp32 per-chunk sum for complex64, fp64 for complex128
#pragma unroll
        for (int j = 0; j < 4; ++j) loc += a[j].x * a[j].x + a[j].y * a[j].y;
        acc += (double)loc;
    }
    const double s = block_sum(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

template <typename T>
__global__ void __launch_bounds__(kReduceThreads)
k_pauli_partial(const typename Vec2<T>::type* __restrict__ psi, GroupSpec gs, uint64_t xmask, uint64_t zmask,
                int ny, double coeff, double* __restrict__ partials)
{
    using V = typename Vec2<T>::type;
    double acc = 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x * 4;
    const uint64_t n = gs.n_groups;
    for (uint64_t g0 = (uint64_t)blockIdx.x * blockDim.x * 4 + threadIdx.x; g0 < n + threadIdx.x; g0 += stride) {
        uint64_t x[4];
        V a[4], b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t g = g0 + (uint64_t)j * blockDim.x;
            if (g < n) {
                x[j] = group_base(g, gs);
                a[j] = psi[x[j]];
                if (xmask) b[j] = psi[x[j] ^ xmask];
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t g = g0 + (uint64_t)j * blockDim.x;
            if (g < n) {
                const double sgn = (__popcll(x[j] & zmask) & 1) ? -1.0 : 1.0;
                const double ar = (double)a[j].x, ai = (double)a[j].y;
                if (xmask == 0) {
                    acc += sgn * (ar * ar + ai * ai);
                } else {
                    const double br = (double)b[j].x, bi = (double)b[j].y;
                    // w = conj(b) * a
                    const double wr = br * ar + bi * ai;
                    const double wi = br * ai - bi * ar;
                    // Re(i^ny * w)
                    double re;
                    switch (ny & 3) {
                    case 0: re = wr; break;
                    case 1: re = -wi; break;
                    case 2: re = -wr; break;
                    default: re = wi; break;
                    }
                    acc += 2.0 * sgn * re;
                }
            }
        }
    }
    const double s = block_sum(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = coeff * s;
}

// kind 1: o(x) = n - 2 pc(x)                           (sum_i Z_i)
// kind 2: o(x) = (n-1) - 2 pc((x ^ (x>>1)) & (2^(n-1)-1))  (sum_i Z_i Z_{i+1})
template <typename T>
__global__ void __launch_bounds__(kReduceThreads)
k_diag_obs_partial(const typename Vec2<T>::type* __restrict__ psi, uint64_t n_amps, int nq, int kind,
                   double coeff, double* __restrict__ partials)
{
    using V = typename Vec2<T>::type;
    double acc = 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x * 4;
    const uint64_t zzmask = nq > 1 ? ((1ull << (nq - 1)) - 1ull) : 0ull;
    for (uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x * 4 + threadIdx.x; i0 < n_amps + threadIdx.x;
         i0 += stride) {
        V a[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t i = i0 + (uint64_t)j * blockDim.x;
            if (i < n_amps) a[j] = psi[i];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t x = i0 + (uint64_t)j * blockDim.x;
            if (x < n_amps) {
                const double o = kind == 1 ? (double)(nq - 2 * (int)__popcll(x))
                                           : (double)((nq - 1) - 2 * (int)__popcll((x ^ (x >> 1)) & zzmask));
                const double ar = (double)a[j].x, ai = (double)a[j].y;
                acc += o * (ar * ar + ai * ai);
            }
        }
    }
    const double s = block_sum(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = coeff * s;
}

struct DiagTerms {
    int32_t nterms;
    double c[kDiagTermsPerPass];
    uint64_t z[kDiagTermsPerPass];
};

// o(x) = sum_k c_k (-1)^{pc(x & z_k)} per amplitude: nothing is staged, so a
// few terms on a state that the last-level cache holds cost the least here
// (diag_terms_direct says where); each further term is a popcount and an add
// for every amplitude, where k_obs_tile pays one per thread and tile.
template <typename T>
__global__ void __launch_bounds__(kReduceThreads)
k_diag_terms_partial(const typename Vec2<T>::type* __restrict__ psi, uint64_t n_amps, DiagTerms terms,
                     double* __restrict__ partials)
{
    using V = typename Vec2<T>::type;
    double acc = 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x * 4;
    for (uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x * 4 + threadIdx.x; i0 < n_amps + threadIdx.x;
         i0 += stride) {
        V a[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t i = i0 + (uint64_t)j * blockDim.x;
            if (i < n_amps) a[j] = psi[i];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t x = i0 + (uint64_t)j * blockDim.x;
            if (x < n_amps) {
                double o = 0.0;
                for (int k = 0; k < terms.nterms; ++k)
                    o += (__popcll(x & terms.z[k]) & 1) ? -terms.c[k] : terms.c[k];
                const double ar = (double)a[j].x, ai = (double)a[j].y;
                acc += o * (ar * ar + ai * ai);
            }
        }
    }
    const double s = block_sum(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// Many Pauli terms in one read of the state (ObsTilePass).  A term's xmask
// lies inside the tile, so both amplitudes of each of its pairs are in the
// workgroup's LDS copy; its zmask's bits outside the tile are one sign per
// tile.  Terms on one xmask (XX and YY of a bond) share the pair product.
// Diagonal terms come from the squares of the amplitudes a thread loaded:
// their Walsh-Hadamard transform over the register bits gives the signed sum
// for each register part of a zmask, after which a term costs one sign and
// one multiply-add per thread and tile instead of one per amplitude.  (Where
// the squares overflow the sums are differences of infinities: not a number,
// while an amplitude weighed by the diagonal's value would give an infinity.
// Weighing them, always or in a branch, made long lists 4 to 7% slower: 29
// qubits complex128, 32 terms 1.60 -> 1.70 ms.)  The
// next tile is loaded into registers while the current one is evaluated.
// A term is one 32-byte scalar load, fetched a term ahead: with its fields in
// separate arrays the loop waited on one load after the other (27 qubits
// complex128, 26 bonds of XX + YY and 53 diagonal terms: 1.03 ms a pass
// against 0.89).  What bounds it: about 20 vector instructions per pair and
// term against 0.34 ms for reading the 2 GiB once.
template <typename T>
__global__ void __launch_bounds__(kObsTileThreads)
k_obs_tile(const typename Vec2<T>::type* __restrict__ psi, uint32_t n_tiles, ObsTilePass ps,
           double* __restrict__ partials)
{
    using V = typename Vec2<T>::type;
    constexpr int R = 1 << kObsRegBits;
    constexpr int kLaneBits = kObsTileBits - kObsRegBits;
    __shared__ V lds[1 << kObsTileBits];
    const uint32_t t = threadIdx.x, na = 1u << ps.tq, half = na >> 1;
    uint64_t toff = 0;
#pragma unroll
    for (int i = 0; i < kLaneBits; ++i)
        if (i < ps.tq) toff |= (uint64_t)((t >> i) & 1u) << ps.q[i];
    uint64_t roff[R];
    roff[0] = 0;
#pragma unroll
    for (int j = 1; j < R; ++j) {
        const int b = __builtin_ctz(j);
        roff[j] = roff[j & (j - 1)] | (kLaneBits + b < ps.tq ? 1ull << ps.q[kLaneBits + b] : 0ull);
    }
    auto base_of = [&](uint32_t tile) {
        uint64_t b = tile;
        for (int k = 0; k < ps.tq; ++k) {
            const int p = ps.q[k];
            b = ((b >> p) << (p + 1)) | (b & ((1ull << p) - 1ull));
        }
        return b;
    };
    V r[R];
    auto load = [&](uint64_t base) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (t + (uint32_t)j * kObsTileThreads < na) r[j] = ldg<true>(psi + (base | toff | roff[j]));
            else r[j].x = r[j].y = T(0);
        }
    };
    double acc = 0.0;
    uint32_t tile = blockIdx.x;
    uint64_t base = base_of(tile);
    load(base);
    for (;;) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const uint32_t l = t + (uint32_t)j * kObsTileThreads;
            if (l < na) lds[l] = r[j];
        }
        if (ps.dstart[R]) {
            double w[R];
#pragma unroll
            for (int j = 0; j < R; ++j) w[j] = (double)r[j].x * (double)r[j].x + (double)r[j].y * (double)r[j].y;
#pragma unroll
            for (int h = 1; h < R; h <<= 1)
#pragma unroll
                for (int j = 0; j < R; ++j)
                    if (!(j & h)) {
                        const double a = w[j], b = w[j | h];
                        w[j] = a + b;
                        w[j | h] = a - b;
                    }
#pragma unroll
            for (int j = 0; j < R; ++j)
                for (int k = ps.dstart[j]; k < ps.dstart[j + 1]; ++k) {
                    const ObsDiagTerm d = ps.diag[k];
                    acc += flip_if(d.c, (uint32_t)__popcll(base & d.z) + (uint32_t)__popc(t & d.zl)) * w[j];
                }
        }
        const uint32_t next = tile + gridDim.x;
        const bool more = next < n_tiles;
        const uint64_t nbase = more ? base_of(next) : 0;
        if (more) load(nbase);
        __syncthreads();
        double wr[R / 2], wi[R / 2];
        uint32_t l[R / 2];
        ObsOffTerm nx = ps.off[0];
        for (int k = 0; k < ps.n_off; ++k) {
            const ObsOffTerm o = nx;
            nx = ps.off[k + 1 < kObsTileOff ? k + 1 : k];
            if (o.first) {
                const uint32_t f = o.f;
                const int p = 31 - __builtin_clz(f);
#pragma unroll
                for (int j = 0; j < R / 2; ++j) {
                    const uint32_t i = t + (uint32_t)j * kObsTileThreads;
                    l[j] = ((i >> p) << (p + 1)) | (i & ((1u << p) - 1u));
                    V a, b;
                    a.x = a.y = b.x = b.y = T(0);
                    if (i < half) {
                        a = lds[l[j]];
                        b = lds[l[j] ^ f];
                    }
                    const double ar = a.x, ai = a.y, br = b.x, bi = b.y;
                    wr[j] = br * ar + bi * ai;  // conj(b) a
                    wi[j] = br * ai - bi * ar;
                }
            }
            double s = 0.0;
            if (o.imag) {
#pragma unroll
                for (int j = 0; j < R / 2; ++j) s += flip_if(wi[j], (uint32_t)__popc(l[j] & o.zl));
            } else {
#pragma unroll
                for (int j = 0; j < R / 2; ++j) s += flip_if(wr[j], (uint32_t)__popc(l[j] & o.zl));
            }
            acc += flip_if(o.c, (uint32_t)__popcll(base & o.z)) * s;
        }
        __syncthreads();  // every read of this tile precedes the next one's writes
        if (!more) break;
        tile = next;
        base = nbase;
    }
    // block sum, fixed order (the tile's LDS is free)
    double* sm = (double*)lds;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if ((t & 63u) == 0) sm[t >> 6] = acc;
    __syncthreads();
    if (t == 0) {
        double s = 0.0;
        for (int w = 0; w < kObsTileThreads / 64; ++w) s += sm[w];
        partials[blockIdx.x] = s;
    }
}

// out[seg] = scale[seg] * sum of partials[seg * seg_len .. +seg_len) (fixed order);
// one block per segment.
__global__ void __launch_bounds__(kReduceThreads)
k_sum_segments(const double* __restrict__ partials, int seg_len, const double* __restrict__ scale,
               double* __restrict__ out)
{
    const double* p = partials + (size_t)blockIdx.x * seg_len;
    double acc = 0.0;
    for (int i = threadIdx.x; i < seg_len; i += blockDim.x) acc += p[i];
    const double s = block_sum(acc);
    if (threadIdx.x == 0) out[blockIdx.x] = scale ? scale[blockIdx.x] * s : s;
}

// --------------------------------------------------------------------------
// launchers
// --------------------------------------------------------------------------
template <typename T>
hipError_t launch_norm_partial(const void* psi, uint64_t n_amps, double* partials, hipStream_t s)
{
    using V = typename Vec2<T>::type;
    const int nb = reduce_grid(n_amps);
    hipLaunchKernelGGL((k_norm_partial<T>), dim3(nb), dim3(kReduceThreads), 0, s, (const V*)psi, n_amps,
                       partials);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_pauli_partial(const void* psi, int n, uint64_t xmask, uint64_t zmask, int ny, double coeff,
                                double* partials, hipStream_t s)
{
    using V = typename Vec2<T>::type;
    GroupSpec gs{};
    if (xmask == 0) {
        gs.n_groups = 1ull << n;
        gs.nins = 0;
    } else {
        gs.n_groups = 1ull << (n - 1);
        gs.nins = 1;
        gs.pos[0] = 63 - __builtin_clzll(xmask);
    }
    gs.set_mask = 0;
    const int nb = reduce_grid(gs.n_groups);
    hipLaunchKernelGGL((k_pauli_partial<T>), dim3(nb), dim3(kReduceThreads), 0, s, (const V*)psi, gs, xmask, zmask,
                       ny, coeff, partials);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_diag_obs_partial(const void* psi, int n, int kind, double coeff, double* partials, hipStream_t s)
{
    using V = typename Vec2<T>::type;
    const uint64_t n_amps = 1ull << n;
    const int nb = reduce_grid(n_amps);
    hipLaunchKernelGGL((k_diag_obs_partial<T>), dim3(nb), dim3(kReduceThreads), 0, s, (const V*)psi, n_amps, n,
                       kind, coeff, partials);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_diag_terms_partial(const void* psi, int n, const double* hcoef, const uint64_t* hz, int nterms,
                                     double* partials, hipStream_t s)
{
    using V = typename Vec2<T>::type;
    DiagTerms terms{};
    if (nterms > kDiagTermsPerPass) return hipErrorInvalidValue;
    terms.nterms = nterms;
    for (int k = 0; k < nterms; ++k) {
        terms.c[k] = hcoef[k];
        terms.z[k] = hz[k];
    }
    const uint64_t n_amps = 1ull << n;
    hipLaunchKernelGGL((k_diag_terms_partial<T>), dim3(reduce_grid(n_amps)), dim3(kReduceThreads), 0, s,
                       (const V*)psi, n_amps, terms, partials);
    return hipGetLastError();
}

int obs_tile_blocks(int n)
{
    const uint64_t tiles = n > kObsTileBits ? 1ull << (n - kObsTileBits) : 1ull;
    return (int)std::min<uint64_t>(tiles, kReduceBlocks);
}

template <typename T>
hipError_t launch_obs_tile(const void* psi, int n, const ObsTilePass& ps, double* partials, hipStream_t s)
{
    using V = typename Vec2<T>::type;
    const uint64_t tiles = 1ull << (n - ps.tq);
    if (ps.tq != std::min(n, kObsTileBits) || tiles >= (1ull << 31)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_obs_tile<T>), dim3(obs_tile_blocks(n)), dim3(kObsTileThreads), 0, s, (const V*)psi,
                       (uint32_t)tiles, ps, partials);
    return hipGetLastError();
}

hipError_t launch_sum_partials(const double* partials, int count, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_sum_segments, dim3(1), dim3(kReduceThreads), 0, s, partials, count, (const double*)nullptr,
                       out);
    return hipGetLastError();
}

hipError_t launch_sum_segments(const double* partials, int seg_len, int n_seg, const double* scale, double* out,
                               hipStream_t s)
{
    if (n_seg <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_sum_segments, dim3(n_seg), dim3(kReduceThreads), 0, s, partials, seg_len, scale, out);
    return hipGetLastError();
}

int reduce_blocks_for(uint64_t n_items) { return reduce_grid(n_items); }

template hipError_t launch_norm_partial<double>(const void*, uint64_t, double*, hipStream_t);
template hipError_t launch_norm_partial<float>(const void*, uint64_t, double*, hipStream_t);
template hipError_t launch_pauli_partial<double>(const void*, int, uint64_t, uint64_t, int, double, double*,
                                                 hipStream_t);
template hipError_t launch_pauli_partial<float>(const void*, int, uint64_t, uint64_t, int, double, double*,
                                                hipStream_t);
template hipError_t launch_diag_obs_partial<double>(const void*, int, int, double, double*, hipStream_t);
template hipError_t launch_diag_obs_partial<float>(const void*, int, int, double, double*, hipStream_t);
template hipError_t launch_diag_terms_partial<double>(const void*, int, const double*, const uint64_t*, int, double*,
                                                      hipStream_t);
template hipError_t launch_diag_terms_partial<float>(const void*, int, const double*, const uint64_t*, int, double*,
                                                     hipStream_t);
template hipError_t launch_obs_tile<double>(const void*, int, const ObsTilePass&, double*, hipStream_t);
template hipError_t launch_obs_tile<float>(const void*, int, const ObsTilePass&, double*, hipStream_t);

}  // namespace svk
