// The device's op lists, layouts, supports and gradient groups against the
// planner's (a host-logic test; no GPU).
//
// The kernels read lists made from the planner's: lane bits as thread bits,
// runs of subset phases as tables, layouts as byte offsets.  Compiled from the
// library's own host source, these are compared here with what the planner's
// lists say, thread by thread: the phase every thread of a sample of tiles
// applies for each op and run, the LDS slot and the state offset of every
// register, the lanes each control selects.  The passes' supports are compared
// with the indices that gates can reach from |0...0>, and with which
// amplitudes earlier passes have stored.
#include "sv_batch.hip"

#include <complex>
#include <cstdio>
#include <random>
#include <set>

using cd = std::complex<double>;

static int errors = 0;
#define CHECK(c, ...) do { if (!(c)) { ++errors; if (errors < 20) { printf("FAIL line %d ", __LINE__); printf(__VA_ARGS__); printf("\n"); } } } while (0)

static long tables, byte_tables[4], lane_tables, list_runs, masked_ops, layouts_seen;

struct Circ {
    int n;
    std::vector<sv_op> ops;
    int n_params = 0;
};

static std::vector<std::vector<double>*> matrices;
static sv_op mk(int gate, std::vector<int> ctl, std::vector<int> tgt, int pidx = -1, double val = 0.3)
{
    sv_op o;
    memset(&o, 0, sizeof o);
    o.gate = gate;
    o.n_controls = (int)ctl.size();
    o.n_targets = (int)tgt.size();
    int k = 0;
    for (int q : ctl) o.qubits[k++] = q;
    for (int q : tgt) o.qubits[k++] = q;
    o.param_index = pidx;
    o.value = val;
    if (gate == SV_U2 || gate == SV_U4) {
        const int d = gate == SV_U2 ? 2 : 4;
        matrices.push_back(new std::vector<double>(2 * d * d, 0.1));
        o.matrix = matrices.back()->data();
    }
    return o;
}

static uint32_t lane_local(const FLayout& L, uint32_t tl)
{
    uint32_t l = 0;
    for (int i = 0; i < kPassLaneBits; ++i)
        if ((tl >> i) & 1u) l |= L.lane_l[i];
    return l;
}

static void check_layouts(const HostTables& H, size_t eb)
{
    const std::vector<DLayout> D = device_layouts(H, eb);
    for (const FCirc& c : H.circs)
        for (int p = 0; p < c.n_pass; ++p) {
            const FPass& fp = H.passes[c.pass_begin + p];
            auto one = [&](int k, int rb) {
                const FLayout& L = H.lays[k];
                std::set<uint32_t> slots;
                for (uint32_t tl = 0; tl < (1u << (c.tq - rb)); ++tl)
                    for (int j = 0; j < (1 << rb); ++j) {
                        uint32_t l = lane_local(L, tl), addr = D[k].reg_b[j];
                        uint64_t g = 0, dg = D[k].reg_g[j];
                        for (int i = 0; i < c.tq - rb; ++i)
                            if ((tl >> i) & 1u) {
                                addr ^= D[k].lane_b[i];
                                dg += D[k].lane_g[i];
                                g |= 1ull << fp.q[L.pos[i]];
                            }
                        for (int r = 0; r < rb; ++r)
                            if ((j >> r) & 1) {
                                l |= 1u << L.pos[c.tq - rb + r];
                                g |= 1ull << fp.q[L.pos[c.tq - rb + r]];
                            }
                        const uint32_t s = l ^ (((l >> 4) ^ (l >> 8) ^ (l >> 12)) & 15u);
                        CHECK(addr == s * eb, "layout %d thread %u register %d: slot %u, not %u", k, tl, j, addr, (unsigned)(s * eb));
                        CHECK(dg == g * eb, "layout %d thread %u register %d: state offset", k, tl, j);
                        CHECK(slots.insert(addr).second && addr < (eb << c.tq), "layout %d: slot %u twice or outside", k, addr);
                    }
                ++layouts_seen;
            };
            if (c.reg)
                for (int k = fp.lay_begin, o = fp.op_begin; ; ++o) {
                    one(k, H.reg_bits);
                    while (o < fp.op_end && H.fops[o].kind != FK_LAYOUT) ++o;
                    if (o >= fp.op_end) break;
                    k = H.fops[o].a;
                }
        }
}

// The thread-index condition of a device op equals the planner's tile-local one.
static void check_lanes(const FOp& f, const FOp& d, const FLayout& L, uint32_t threads)
{
    if (f.cml) ++masked_ops;
    for (uint32_t tl = 0; tl < threads; ++tl) {
        const uint32_t l = lane_local(L, tl);
        CHECK(((l & f.cml) == f.cml) == ((tl & d.cml) == d.cml), "kind %d: lanes of the controls", f.kind);
        if ((f.kind == FK_DIAG || f.kind == FK_PHASE) && f.ka < 0)
            CHECK(((l >> f.a) & 1u) == ((tl >> d.a) & 1u), "kind %d: lane of the target", f.kind);
        if (f.kind == FK_PAIRC && f.kb < 0) CHECK(((l >> f.b) & 1u) == ((tl >> d.b) & 1u), "lane of the selector");
    }
}

static void check_ops(HostTables& H, std::mt19937_64& rng)
{
    std::vector<FPass> before = H.passes;
    DeviceOps D = device_ops(H);
    // a phase for every coefficient pair, and the tables as the kernel fills them
    std::vector<double> coef(D.coef_total + 2);
    std::uniform_real_distribution<double> U(0, 6.283);
    for (const FOp& f : H.fops)
        if (f.kind == FK_PHASE) {
            const double th = U(rng);
            coef[f.coef] = cos(th);
            coef[f.coef + 1] = sin(th);
        }
    for (const FRunTab& t : D.tabs) {
        CHECK(t.dst >= H.coef_total && t.dst + 2 * t.n <= D.coef_total, "table outside the coefficients");
        for (int e = 0; e < t.n; ++e) {
            cd z = 1;
            for (int k = t.begin; k < t.end; ++k)
                if (((uint32_t)e & D.members[k].mask) == D.members[k].mask)
                    z *= cd(coef[D.members[k].coef], coef[D.members[k].coef + 1]);
            coef[t.dst + 2 * e] = z.real();
            coef[t.dst + 2 * e + 1] = z.imag();
        }
    }
    auto val = [&](int c) { return cd(coef[c], coef[c + 1]); };
    for (const FCirc& c : H.circs)
        for (int p = 0; p < c.n_pass; ++p) {
            const FPass &pf = before[c.pass_begin + p], &pd = H.passes[c.pass_begin + p];
            if (!c.reg) continue;
            const uint32_t threads = 1u << (c.tq - H.reg_bits);
            int lay = pf.lay_begin, d = pd.op_begin;
            for (int o = pf.op_begin; o < pf.op_end;) {
                const FOp& f = H.fops[o];
                if (d >= pd.op_end) {
                    CHECK(false, "device list ends early");
                    break;
                }
                const FOp& g = D.ops[d++];
                if (f.kind == FK_LAYOUT) {
                    CHECK(g.kind == FK_LAYOUT && g.a == f.a, "layout marker");
                    lay = f.a;
                    ++o;
                    continue;
                }
                if (g.kind != FK_PRUN) {
                    CHECK(g.kind == f.kind && g.coef == f.coef && g.ka == f.ka && g.kb == f.kb && g.cmk == f.cmk, "op %d", o);
                    if (f.kind == FK_PHASE && f.kb == 2 && (o == pf.op_begin || H.fops[o - 1].kb != 2)) ++list_runs;
                    check_lanes(f, g, H.lays[lay], threads);
                    ++o;
                    continue;
                }
                // a run as tables: members [o, e)
                int e = o;
                while (H.fops[e].kind == FK_PHASE && H.fops[e].kb == 2) ++e;
                CHECK(H.fops[e].kind == FK_PHASE && H.fops[e].kb == 3, "end of a run");
                ++e;
                ++tables;
                for (int k = 0; k < 4; ++k) byte_tables[k] += (g.b >> k) & 1;
                lane_tables += g.kb != 0;
                for (int s = 0; s < 64; ++s) {
                    const int tile = s == 0 ? 0 : s == 1 ? c.n_tiles - 1 : (int)(rng() % (uint64_t)c.n_tiles);
                    cd tz = 1;
                    int off = 0;
                    for (uint32_t m = (uint32_t)g.b; m; m &= m - 1u, off += 512)
                        tz *= val(g.coef + off + 2 * (int)(((uint32_t)tile >> (8 * __builtin_ctz(m))) & 255u));
                    for (uint32_t tl = 0; tl < threads; ++tl) {
                        const uint32_t l = lane_local(H.lays[lay], tl);
                        cd ref = 1;
                        for (int k = o; k < e; ++k) {
                            const FOp& q = H.fops[k];
                            const uint32_t lc = q.cml & ~(1u << q.a);
                            if (((uint32_t)tile & (uint32_t)q.b) == (uint32_t)q.b && (l & lc) == lc) ref *= val(q.coef);
                        }
                        const cd z = g.kb ? tz * val(g.coef + off + 2 * (int)tl) : tz;
                        CHECK(std::abs(z - ref) < 1e-12, "run at op %d, tile %d, thread %u", o, tile, tl);
                    }
                }
                // applied to the amplitudes holding the target
                const uint32_t cmk = f.ka >= 0 ? 1u << f.ka : 0u;
                CHECK(g.cmk == cmk && g.ka == f.ka, "target register of a run");
                for (uint32_t tl = 0; tl < threads; ++tl)
                    CHECK(((tl & g.cml) == g.cml) == (f.ka >= 0 || ((lane_local(H.lays[lay], tl) >> f.a) & 1u)), "target lane of a run");
                o = e;
            }
            CHECK(d == pd.op_end, "device list has %d ops more", pd.op_end - d);
        }
}

// Indices reachable from |0...0> and stored amplitudes, pass by pass.
static void check_supports(const Circ& C, int dtype, const HostTables& H)
{
    const FCirc& c = H.circs[0];
    const int n = C.n;
    std::vector<BOp> ops;
    int max_q = 1;
    for (size_t i = 0; i < C.ops.size(); ++i) {
        BOp o;
        CHECK(validate(n, C.ops[i], C.n_params, (int)i, &o) == SV_OK, "validate");
        max_q = std::max(max_q, o.nc + o.nt);
        ops.push_back(o);
    }
    std::vector<std::vector<int>> pops;
    std::vector<uint64_t> pq;
    schedule(n, c.tq, std::max(0, std::min(dtype == SV_C128 ? 3 : 4, c.tq - max_q)), ops, pops, pq);
    CHECK((int)pops.size() == c.n_pass, "passes");
    const uint64_t N = 1ull << n;
    std::vector<char> reach(N, 0), stored(N, 0);
    reach[0] = 1;
    for (int p = 0; p < c.n_pass; ++p) {
        const FPass& fp = H.passes[c.pass_begin + p];
        const uint64_t out = ~fp.support;
        for (uint64_t x = 0; x < N; ++x) {
            CHECK(!reach[x] || !(x & out), "pass %d: reachable index outside the support", p);
            if (p && !(x & out)) CHECK(stored[x], "pass %d loads an amplitude that no pass stored", p);
        }
        for (uint64_t x = 0; x < N; ++x)
            if (p + 1 == c.n_pass || !(x & fp.free_mask & out)) stored[x] = 1;
        for (int i : pops[p]) {
            const BOp& o = ops[i];
            uint64_t cm = 0, tm = 0;
            for (int j = 0; j < o.nc; ++j) cm |= 1ull << o.q[j];
            for (int j = o.nc; j < o.nc + o.nt; ++j) tm |= 1ull << o.q[j];
            if (diag_gate(o.gate)) continue;
            std::vector<char> was = reach;
            for (uint64_t x = 0; x < N; ++x) {
                if (!was[x] || (x & cm) != cm) continue;
                uint64_t s = tm;  // every pattern of the target bits
                for (;; s = (s - 1) & tm) {
                    reach[(x & ~tm) | s] = 1;
                    if (!s) break;
                }
            }
        }
    }
    for (uint64_t x = 0; x < N; ++x) CHECK(stored[x], "amplitude never stored");
}

static void check_groups(const HostTables& H0)
{
    HostTables H = H0;
    std::vector<sv_batch_s::GradGroup> G;
    CHECK(group_gradients(H, G) == SV_OK, "groups: %s", sv_last_error());
    const FCirc& c = H0.circs[0];
    const int slots = (int)H0.slot_param.size();
    std::vector<int> number(slots, -1);
    size_t level = c.n_pass + 1, gi = 0;
    std::set<int> used;
    for (int p = c.n_pass - 1; p >= 0; --p) {
        const size_t at = (size_t)(2 * c.n_pass - p);  // the pass's level
        while (gi < G.size() && at >= G[gi].level_end) {
            CHECK(G[gi].level_end >= level, "levels");
            level = G[gi].level_end;
            ++gi;
            used.clear();
        }
        CHECK(gi < G.size(), "pass %d in no group", p);
        const FPass& fp = H0.passes[c.pass_begin + p];
        for (int o = fp.rop_begin; o < fp.rop_end; ++o)
            for (int w = 0; w < 2; ++w) {
                const FOp &a = H0.fops[o], &b = H.fops[o];
                if (w == 1 && a.kind != FK_RFUSE) continue;
                const int s = w ? a.b : a.slot, l = w ? b.b : b.slot;
                if (s < 0) {
                    CHECK(l == s, "slot appeared");
                    continue;
                }
                const int k = G[gi].slot_begin + l;
                CHECK(l >= 0 && k < G[gi].slot_end && used.insert(l).second, "slot %d in group %zu", l, gi);
                CHECK((l + 1) * (int64_t)c.n_tiles <= H.g_total, "partials outside the array");
                CHECK(H.g_off[k] == c.g_part_begin + l * (int64_t)c.n_tiles && H.g_cnt[k] == c.n_tiles, "offset");
                CHECK(H.slot_param[k] == H0.slot_param[s] && H.slot_scale[k] == H0.slot_scale[s], "parameter");
                number[s] = k;
            }
    }
    CHECK(G.back().level_end == (size_t)(2 * c.n_pass + 1) && G.back().slot_end == slots && G[0].slot_begin == 0, "ends");
    for (size_t g = 1; g < G.size(); ++g) CHECK(G[g].slot_begin == G[g - 1].slot_end, "groups adjoin");
    for (size_t k = 0; k < H0.csr_col.size(); ++k) CHECK(H.csr_col[k] == number[H0.csr_col[k]], "sum order");
    printf("  groups %zu slots %d partials %.1f MiB (all at once %.1f)\n", G.size(), slots, H.g_total * 8.0 / (1 << 20),
           H0.g_total * 8.0 / (1 << 20));
}

static bool compile(const Circ& C, int dtype, int tile, int apt, int grad, HostTables& H)
{
    sv_batch_circuit bc{C.n, (int)C.ops.size(), C.ops.data(), C.n_params, 1};
    sv_batch_opts op{tile, apt, 0, grad};
    const sv_status rc = compile_batch(&bc, 1, dtype, &op, H);
    CHECK(rc == SV_OK, "compile: %s", sv_last_error());
    return rc == SV_OK;
}

// Controlled phases onto a few targets; nc controls anywhere (far: all above the tile).
static Circ phases(std::mt19937_64& rng, int n, int count, int max_nc, int n_params)
{
    Circ C;
    C.n = n;
    C.n_params = n_params;
    for (int q = 0; q < n; ++q) C.ops.push_back(mk(SV_H, {}, {q}));
    for (int r = 0; r < 4; ++r) {
        const int t = (int)(rng() % n);
        for (int i = 0; i < count; ++i) {
            std::vector<int> ctl;
            const int nc = (int)(rng() % (max_nc + 1));
            while ((int)ctl.size() < nc) {
                const int q = (int)(rng() % n);
                if (q != t && std::find(ctl.begin(), ctl.end(), q) == ctl.end()) ctl.push_back(q);
            }
            if (n_params && rng() % 2) C.ops.push_back(mk(SV_PHASE, ctl, {t}, (int)(rng() % n_params)));
            else C.ops.push_back(mk(rng() % 3 ? SV_PHASE : SV_T, ctl, {t}));
        }
        C.ops.push_back(mk(SV_H, {}, {t}));
    }
    return C;
}

static Circ qft(int n)
{
    Circ C;
    C.n = n;
    for (int j = n - 1; j >= 0; --j) {
        C.ops.push_back(mk(SV_H, {}, {j}));
        for (int c = j - 1; c >= 0; --c) C.ops.push_back(mk(SV_PHASE, {c}, {j}));
    }
    return C;
}

// Two-control phases whose controls lie in chosen qubits, onto one target.
static Circ pairs_of(int n, int t, std::vector<std::pair<int, int>> ctl)
{
    Circ C;
    C.n = n;
    C.ops.push_back(mk(SV_H, {}, {t}));
    for (auto [a, b] : ctl) C.ops.push_back(mk(SV_PHASE, {a, b}, {t}));
    for (int q = 0; q < n; ++q)
        if (q != t) C.ops.push_back(mk(SV_PHASE, {q}, {t}));
    return C;
}

static Circ hea(int n, int layers)
{
    Circ C;
    C.n = n;
    C.n_params = 2 * n * layers;
    int p = 0;
    for (int l = 0; l < layers; ++l) {
        for (int q = 0; q < n; ++q) {
            C.ops.push_back(mk(SV_RY, {}, {q}, p++));
            C.ops.push_back(mk(SV_RZ, {}, {q}, p++));
        }
        for (int q = 0; q + 1 < n; ++q) C.ops.push_back(mk(SV_X, {q}, {q + 1}));
    }
    return C;
}

static Circ mixed(std::mt19937_64& rng, int n, int count, int n_params)
{
    Circ C;
    C.n = n;
    C.n_params = n_params;
    const int one[] = {SV_X, SV_Y, SV_Z, SV_H, SV_S, SV_T, SV_RX, SV_RY, SV_RZ, SV_PHASE, SV_U2};
    for (int i = 0; i < count; ++i) {
        std::vector<int> q(n);
        for (int k = 0; k < n; ++k) q[k] = k;
        std::shuffle(q.begin(), q.end(), rng);
        const int r = (int)(rng() % 13);
        if (r == 11) C.ops.push_back(mk(SV_SWAP, {}, {q[0], q[1]}));
        else if (r == 12) C.ops.push_back(mk(SV_U4, {}, {q[0], q[1]}));
        else {
            const int nc = (int)(rng() % 3), g = one[r];
            const bool par = n_params && (g == SV_RX || g == SV_RY || g == SV_RZ || g == SV_PHASE) && rng() % 2;
            C.ops.push_back(mk(g, {q.begin() + 1, q.begin() + 1 + nc}, {q[0]}, par ? (int)(rng() % n_params) : -1));
        }
    }
    return C;
}

int main()
{
    std::mt19937_64 rng(11);
    for (int dt : {SV_C128, SV_C64}) {
        const size_t eb = dt == SV_C128 ? 16 : 8;
        struct Shape {
            int tile, apt;
        };
        for (Shape s : {Shape{5, 8}, Shape{6, 16}, Shape{10, 16}, Shape{12, 16}})
            for (int grad : {0, 1})
                for (int n : {9, 17, 23, 30}) {
                    if (n == 30 && s.tile < 10) continue;  // too many work items for a batch
                    for (int which = 0; which < 4; ++which) {
                        const Circ C = which == 0 ? phases(rng, n, 40, 3, 6) : which == 1 ? qft(n) : which == 2 ? mixed(rng, n, 150, 8) : phases(rng, n, 30, 1, 0);
                        HostTables H;
                        if (!compile(C, dt, s.tile, s.apt, grad, H)) continue;
                        check_layouts(H, eb);
                        check_ops(H, rng);
                    }
                }
        for (Shape s : {Shape{5, 8}, Shape{6, 16}, Shape{8, 16}})
            for (int k = 0; k < 12; ++k) {
                const int n = 9 + k % 4;
                Circ C = k % 3 == 0 ? qft(n) : mixed(rng, n, 10 + 10 * k, 0);
                HostTables H;
                if (compile(C, dt, s.tile, s.apt, 0, H)) check_supports(C, dt, H);
            }
        for (int n : {6, 16, 24, 26})
            for (int layers : {1, 6, 14}) {
                HostTables H;
                if (compile(hea(n, layers), dt, 10, 16, 1, H)) check_groups(H);
            }
        for (int k = 0; k < 6; ++k) {
            HostTables H;
            if (compile(mixed(rng, 20 + k, 400, 30), dt, 10, 16, 1, H)) check_groups(H);
        }
    }
    // controls in the second byte of the tile index, alone and with the first (tile: qubits 0 to 4)
    for (bool across : {false, true}) {
        const Circ C = pairs_of(21, 3, across ? std::vector<std::pair<int, int>>{{14, 15}, {8, 15}, {16, 20}}
                                              : std::vector<std::pair<int, int>>{{14, 15}, {5, 9}, {16, 20}});
        HostTables H;
        if (!compile(C, SV_C128, 5, 8, 0, H)) continue;
        const long t0 = tables, l0 = list_runs;
        check_ops(H, rng);
        CHECK(across ? list_runs > l0 : tables > t0 && list_runs == l0, "form of a run %s two bytes", across ? "across" : "within");
    }
    printf("tables %ld (bytes %ld %ld %ld %ld, lanes %ld) list runs %ld masked ops %ld layouts %ld\n", tables,
           byte_tables[0], byte_tables[1], byte_tables[2], byte_tables[3], lane_tables, list_runs, masked_ops, layouts_seen);
    CHECK(byte_tables[0] && byte_tables[1] && byte_tables[2] && lane_tables && list_runs && masked_ops && layouts_seen, "a form is not exercised");
    printf("%s (%d errors)\n", errors ? "FAILED" : "all ok", errors);
    return errors ? 1 : 0;
}
