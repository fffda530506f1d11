// runs_host.cpp -- the run-based replay and the listing of requests
// (csrc/pc_runs.h) on the CPU: the wavefront is a structure of 64 lanes, LDS
// and device memory are arrays with bounds checks; ids and weak links come
// from a plain map.  Built and driven by test_runs_cpu.py.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <random>
#include <type_traits>
#include <unordered_map>
#include <vector>

#define PC_RUNS_FN inline

namespace {
constexpr int kLanes = 64;
template <class T>
struct V {
    T v[kLanes];
};
template <class T, class S, class F>
auto zip(const V<T> &a, const V<S> &b, F f) {
    V<decltype(f(a.v[0], b.v[0]))> r;
    for (int i = 0; i < kLanes; ++i) r.v[i] = f(a.v[i], b.v[i]);
    return r;
}
template <class T>
V<T> splat(T x) {
    V<T> r;
    for (int i = 0; i < kLanes; ++i) r.v[i] = x;
    return r;
}
#define PC_OP(op)                                                                                        \
    template <class T>                                                                                   \
    auto operator op(const V<T> &a, const V<T> &b) {                                                     \
        return zip(a, b, [](T x, T y) { return T(x op y); });                                            \
    }                                                                                                    \
    template <class T, class S>                                                                          \
    auto operator op(const V<T> &a, S b) -> V<T> {                                                       \
        return zip(a, splat<T>((T)b), [](T x, T y) { return T(x op y); });                               \
    }
PC_OP(+) PC_OP(-) PC_OP(&) PC_OP(|) PC_OP(*)
#define PC_CMP(op)                                                                                       \
    template <class T>                                                                                   \
    V<bool> operator op(const V<T> &a, const V<T> &b) {                                                  \
        return zip(a, b, [](T x, T y) { return x op y; });                                               \
    }                                                                                                    \
    template <class T, class S>                                                                          \
    V<bool> operator op(const V<T> &a, S b) {                                                            \
        return zip(a, splat<T>((T)b), [](T x, T y) { return x op y; });                                  \
    }
PC_CMP(<) PC_CMP(>) PC_CMP(<=) PC_CMP(>=) PC_CMP(==) PC_CMP(!=)
template <class T>
V<T> operator<<(const V<T> &a, int s) { return zip(a, a, [s](T x, T) { return T(x << s); }); }
template <class T>
V<T> operator>>(const V<T> &a, int s) { return zip(a, a, [s](T x, T) { return T(x >> s); }); }
V<int64_t> operator-(const V<int64_t> &a) { return zip(a, a, [](int64_t x, int64_t) { return -x; }); }

uint32_t *g_lds;
int64_t g_lds_words;
[[noreturn]] void die(const char *what) {
    std::fprintf(stderr, "runs_host: %s\n", what);
    std::abort();
}
void check(const uint32_t *p) {
    if (p < g_lds || p >= g_lds + g_lds_words) die("LDS access out of range");
}

// Device memory of the analysis; a read of `before` runs the hook first.
struct Region {
    const uint32_t *p;
    size_t n;
};
std::vector<Region> g_mem;
std::function<void()> g_hook;
const uint32_t *g_hook_at;
void check_mem(const uint32_t *p, size_t words = 1) {
    for (const Region &r : g_mem)
        if (p >= r.p && p + words <= r.p + r.n) return;
    die("device memory access out of range");
}

struct HostWave {
    using vu = V<uint32_t>;
    using vl = V<int64_t>;
    using vb = V<bool>;
    using Lds = uint32_t *;
    vu lane() const {
        vu r;
        for (int i = 0; i < kLanes; ++i) r.v[i] = (uint32_t)i;
        return r;
    }
    vu vu0(uint32_t x) const { return splat<uint32_t>(x); }
    vl vl0(int64_t x) const { return splat<int64_t>(x); }
    static void sync() {}
    static uint64_t ballot(const vb &b) {
        uint64_t m = 0;
        for (int i = 0; i < kLanes; ++i) m |= (uint64_t)b.v[i] << i;
        return m;
    }
    static vb of_mask(uint64_t m) {
        vb r;
        for (int i = 0; i < kLanes; ++i) r.v[i] = (m >> i) & 1u;
        return r;
    }
    static int popc(uint64_t m) { return __builtin_popcountll(m); }
    static int ffs(uint64_t m) {
        if (!m) die("first bit of an empty mask");
        return __builtin_ctzll(m);
    }
    static int clz(uint64_t m) { return __builtin_clzll(m); }
    static uint32_t rdl(const vu &v, int l) {
        if (l < 0 || l >= kLanes) die("lane out of range");
        return v.v[l];
    }
    static int64_t rdl64(const vl &v, int l) { return v.v[l]; }
    template <class T>
    static V<T> sel(const vb &m, const V<T> &a, const V<T> &b) {
        V<T> r;
        for (int i = 0; i < kLanes; ++i) r.v[i] = m.v[i] ? a.v[i] : b.v[i];
        return r;
    }
    template <class T>
    static V<T> vmin(const V<T> &a, const V<T> &b) { return zip(a, b, [](T x, T y) { return x < y ? x : y; }); }
    template <class T>
    static V<T> vmax(const V<T> &a, const V<T> &b) { return zip(a, b, [](T x, T y) { return x > y ? x : y; }); }
    static vl vmax(const vl &a, int64_t b) { return vmax(a, splat<int64_t>(b)); }
    static vu scan(const vu &a) {
        vu r = a;
        for (int i = 1; i < kLanes; ++i) r.v[i] += r.v[i - 1];
        return r;
    }
    static uint32_t wsum(const vu &a) { return scan(a).v[63]; }
    static uint32_t wmax(const vu &a) {
        uint32_t m = 0;
        for (uint32_t x : a.v) m = x > m ? x : m;
        return m;
    }
    static int64_t wmax64(const vl &a) {
        int64_t m = a.v[0];
        for (int64_t x : a.v) m = x > m ? x : m;
        return m;
    }
    static vu mbcnt(uint64_t m) {
        vu r;
        for (int i = 0; i < kLanes; ++i) r.v[i] = (uint32_t)__builtin_popcountll(m & ((1ull << i) - 1));
        return r;
    }
    static vl widen(const vu &a) {
        vl r;
        for (int i = 0; i < kLanes; ++i) r.v[i] = (int64_t)a.v[i];
        return r;
    }
    static vl mul_shr16(const vl &a, int64_t w) {
        return zip(a, a, [w](int64_t x, int64_t) { return (int64_t)(((__int128)x * w) >> 16); });
    }
    static vl mul_sat62(const vl &a, uint32_t b) {
        return zip(a, a, [b](int64_t x, int64_t) {
            const __int128 v = (__int128)x * b;
            return v > ((__int128)1 << 62) ? (int64_t)1 << 62 : (int64_t)v;
        });
    }
    template <class T>
    static T hold(const T &x) { return x; }
    static uint32_t uni(const vu &v) { return v.v[0]; }
    static uint64_t udiv(uint64_t a, uint64_t b) { return a / b; }
    static vu ld(const uint32_t *p, const vu &at) {
        vu r;
        for (int i = 0; i < kLanes; ++i) {
            check(p + at.v[i]);
            r.v[i] = p[at.v[i]];
        }
        return r;
    }
    static void st(const vb &m, uint32_t *p, const vu &at, const vu &x) {
        for (int i = 0; i < kLanes; ++i)
            if (m.v[i]) {
                check(p + at.v[i]);
                p[at.v[i]] = x.v[i];
            }
    }
    static void st_all(uint32_t *p, const vu &at, const vu &x) { st(splat(true), p, at, x); }
    template <int N>
    void st1(uint32_t *p, uint32_t at, uint32_t *scratch, uint32_t x, uint32_t y, uint32_t z) {
        check(scratch + 64 * N - 1);
        const uint32_t v[3] = {x, y, z};
        for (int i = 0; i < N; ++i) {
            check(p + at + 64 * i);
            p[at + 64 * i] = v[i];
        }
    }
    static vu setlane(vu a, int l, uint32_t x) {
        if (l < 0 || l >= kLanes) die("lane out of range");
        a.v[l] = x;
        return a;
    }
    static vu ld_if(const vb &m, const uint32_t *p, const vu &at) {
        vu r = splat<uint32_t>(0);
        for (int i = 0; i < kLanes; ++i)
            if (m.v[i]) {
                check(p + at.v[i]);
                r.v[i] = p[at.v[i]];
            }
        return r;
    }
    uint32_t ld1(const uint32_t *p, uint32_t at) const {
        check(p + at);
        return p[at];
    }
    static vu mad01(const vu &a, uint32_t b, const vu &c) {
        for (uint32_t x : a.v)
            if (x > 1) die("mad01 factor");
        return zip(a, c, [b](uint32_t x, uint32_t z) { return x * b + z; });
    }
    static vu next_lane(const vu &a) {
        vu r;
        for (int i = 0; i < kLanes; ++i) r.v[i] = a.v[(i + 1) % kLanes];
        return r;
    }
    static vu gld(const vb &m, const uint32_t *p, const vu &at) {
        if (p == g_hook_at && g_hook) g_hook();
        vu r = splat<uint32_t>(0);
        for (int i = 0; i < kLanes; ++i)
            if (m.v[i]) {
                check_mem(p + at.v[i]);
                r.v[i] = p[at.v[i]];
            }
        return r;
    }
    static void gst2(const vb &m, uint32_t *p, const vu &at, const vu &x, const vu &y) {
        for (int i = 0; i < kLanes; ++i)
            if (m.v[i]) {
                uint32_t *q = p + 2 * (size_t)at.v[i];
                check_mem(q, 2);
                q[0] = x.v[i];
                q[1] = y.v[i];
            }
    }
    static void gor_bit(const vb &m, uint32_t *p, const vu &i) {
        for (int k = 0; k < kLanes; ++k)
            if (m.v[k]) {
                check_mem(p + (i.v[k] >> 5));
                p[i.v[k] >> 5] |= 1u << (i.v[k] & 31);
            }
    }
    static vb bit(const vu &w, const vu &i) {
        return zip(w, i, [](uint32_t x, uint32_t k) { return ((x >> (k & 31)) & 1u) != 0; });
    }
    static uint32_t keep(uint32_t x) { return x; }
    static vl mad64(const vu &a, int32_t b, const vl &c) {
        return zip(a, c, [b](uint32_t x, int64_t z) { return (int64_t)x * b + z; });
    }
    static bool likely(bool x) { return x; }
    static bool unlikely(bool x) { return x; }
};
}  // namespace

#include "pc_runs.h"

namespace {

// A trace on the key buffer (group to tick: of the one that is replayed).
struct TraceIn {
    const int64_t *off;
    int64_t n_req;
    const uint8_t *group, *contract;
    const uint32_t *prefix;
    const int64_t *tick;
};
struct Analysis {
    std::vector<uint32_t> id, start, weak, cuts;
    std::vector<pcr::RunPiece> piece;
    std::vector<pcr::RunReq> req;      // of the trace that is replayed
    bool left = false;                 // it is not for this form
};

// Analysis of a key buffer that `ts` read, their requests listed in this
// order; ts[main] is replayed.  With `interleave` (a seed) the first pass lists
// another request ahead of every step of 64 blocks of one, as other wavefronts
// may at any time.
Analysis analyse(const uint64_t *keys, int64_t n, const std::vector<TraceIn> &ts, size_t main, int interleave) {
    Analysis A;
    const size_t words = (size_t)(n + 31) / 32;
    A.id.resize(n);
    A.start.assign(words, 0);
    A.weak.assign(words, 0);
    A.cuts.assign(words, 0);
    A.piece.resize(n);
    auto bit = [](const std::vector<uint32_t> &b, int64_t i) { return (b[i >> 5] >> (i & 31)) & 1u; };
    std::unordered_map<uint64_t, uint32_t> first;
    for (int64_t i = 0; i < n; ++i) A.id[i] = first.emplace(keys[i], (uint32_t)i).first->second;
    for (const TraceIn &t : ts)
        for (int64_t r = 0; r < t.n_req; ++r)
            pcr::request_marks(t.off[r], t.off[r + 1] - t.off[r], r + 1 == t.n_req, n,
                               [&](int64_t at) { A.start[at >> 5] |= 1u << (at & 31); });
    for (int64_t i = 0; i < n; ++i)
        if (i == 0 || bit(A.start, i) || A.id[i - 1] + 1 != A.id[i]) A.weak[A.id[i] >> 5] |= 1u << (A.id[i] & 31);
    for (uint32_t &x : A.id) x |= pcr::kRunsResolved;

    pcr::RunsBuf B;
    B.id = A.id.data();
    B.weak = A.weak.data();
    B.cuts = A.cuts.data();
    B.start = A.start.data();
    B.piece = (uint32_t *)A.piece.data();
    g_mem = {{B.id, A.id.size()}, {B.weak, words}, {B.cuts, words}, {B.start, words}, {B.piece, 2 * A.piece.size()}};
    HostWave wv;
    bool cut = false;
    std::vector<uint8_t> left(ts.size(), 0);
    auto list = [&](auto again, size_t t, int64_t r) {
        uint32_t lds[128];
        uint32_t *const outer = g_lds;
        const int64_t outer_words = g_lds_words;
        g_lds = lds;
        g_lds_words = 128;
        const auto L = pcr::list_request<HostWave, decltype(again)::value>(
            wv, B, (uint32_t)ts[t].off[r], (uint32_t)(ts[t].off[r + 1] - ts[t].off[r]), lds);
        g_lds = outer;
        g_lds_words = outer_words;
        cut = cut || L.cut;
        if (L.left) left[t] = 1;
        return L;
    };
    // every request once; the hook lists one that has not begun yet
    std::vector<std::pair<size_t, int64_t>> todo;
    for (size_t t = ts.size(); t-- > 0;)
        for (int64_t r = ts[t].n_req; r-- > 0;) todo.push_back({t, r});
    std::mt19937 rng(interleave);
    auto list_one = [&](size_t k) {
        const auto q = todo[k];
        todo.erase(todo.begin() + (int64_t)k);
        list(std::false_type(), q.first, q.second);
    };
    bool nested = false;
    g_hook_at = B.weak;
    if (interleave)
        g_hook = [&] {
            if (nested || todo.empty()) return;
            nested = true;
            list_one(rng() % todo.size());
            nested = false;
        };
    while (!todo.empty()) list_one(todo.size() - 1);
    g_hook = nullptr;
    std::unordered_map<uint32_t, int> seen;
    for (int pass = cut ? 1 : 0; pass >= 0; --pass)      // (without cuts the same lists again)
        for (size_t t = 0; t < ts.size(); ++t)
            for (int64_t r = 0; r < ts[t].n_req && !left[t]; ++r) {
                const auto L = cut ? list(std::true_type(), t, r) : list(std::false_type(), t, r);
                if (pass > 0 || t != main) continue;
                const TraceIn &T = ts[t];
                const bool before = !seen.emplace(T.prefix[r], 1).second;
                A.req.push_back({(uint32_t)(T.off[r + 1] - T.off[r]),
                                 T.group[r] | ((uint32_t)T.contract[r] << 8) | (before ? 1u << 16 : 0u) |
                                     L.np << 24,
                                 T.prefix[r], (uint32_t)(T.tick ? T.tick[r] - (r ? T.tick[r - 1] : 0) : r ? 1 : 0),
                                 (uint32_t)T.off[r], L.nn, {}});
            }
    A.left = left[main] != 0;
    return A;
}

// All requests; false if a window was too small.
template <class X>
bool all_requests(X &R, const Analysis &A, int64_t n, int64_t n_prefix, int32_t *pr) {
    std::vector<uint8_t> adm(n_prefix + 1, 0);
    for (int64_t r = 0; r < n; ++r) {
        const pcr::RunReq &q = A.req[r];
        V<uint32_t> id = splat<uint32_t>(0), len = splat<uint32_t>(0);
        const uint32_t np = q.info >> 24;
        for (uint32_t i = 0; i < 64 && np > 0; ++i) {
            const pcr::RunPiece &p = A.piece[q.ko + (i < np ? i : 0)];
            id.v[i] = p.id;
            len.v[i] = p.len;
        }
        adm[q.prefix] = R.request((uint32_t)r, q, id, len, adm[q.prefix] != 0);
        if (R.over) return false;
        if ((r + 1) % 100 == 0) R.flush();
        if (pr) {
            pr[4 * r] = R.last_h;
            pr[4 * r + 1] = R.last_m;
            pr[4 * r + 2] = R.last_e;
            pr[4 * r + 3] = R.last_o;
        }
    }
    return true;
}

template <class X>
void results(X &R, const pcr::RunParams &P, int64_t *gs, int64_t *is) {
    R.flush();
    const auto dend = R.raw_debt();
    for (int g = 0; g < P.G; ++g) {
        const int64_t probe = R.c_probe.v[g], hit = R.c_hit.v[g], dup = R.c_dup.v[g];
        const int64_t f[17] = {R.c_req.v[g], probe, hit, probe - hit, probe - hit - dup, R.c_evw.v[g], R.c_evc.v[g],
                               R.c_promo.v[g], R.c_gated.v[g], R.c_orph.v[g], dup, R.c_trunc.v[g],
                               P.n_req ? dend.v[g] : 0, R.d_max.v[g], R.d_sum.v[g], (int64_t)R.res.v[g],
                               (int64_t)R.res_max.v[g]};
        for (int k = 0; k < 17; ++k) gs[17 * g + k] = f[k];
    }
    int64_t ev = 0;
    for (int64_t x : R.c_evw.v) ev += x;
    const int64_t f[7] = {ev, R.c_moves.v[0], R.c_reins.v[0], R.c_ghits.v[0], R.c_gins.v[0], R.resident, R.rmax.v[0]};
    for (int k = 0; k < 7; ++k) is[k] = f[k];
}

template <int kPol, bool kK1>
bool replay_in(const Analysis &A, const pcr::RunParams &P, int64_t n_prefix, int64_t *gs, int64_t *is, int32_t *pr) {
    std::vector<uint32_t> lds(pcr::runs_lds_bytes(kPol, P.win, 0) / 4, 0xDEADBEEFu);
    g_lds = lds.data();
    g_lds_words = (int64_t)lds.size();
    HostWave wv;
    pcr::RunReplay<HostWave, kPol, kK1> R(P, wv, lds.data());
    if (!all_requests(R, A, P.n_req, n_prefix, pr)) return false;
    results(R, P, gs, is);
    return true;
}

}  // namespace

// The oracle's signature; `window` overrides the windows' size (0 and -1: the
// planner's, the widest).  The key buffer has n_keys keys; off2 (or null): a
// second trace that reads it, listed behind the first, or ahead of it
// (ahead2).  Returns 1 when the replay leaves the
// instance, 2 when the analysis does.
extern "C" int runs_host_replay(const uint64_t *keys, const int64_t *off, const uint8_t *group,
                                const uint8_t *contract, const uint32_t *prefix, const int64_t *tick, int64_t n_req,
                                int32_t G, int64_t n_prefix, int32_t policy, int64_t C, int32_t flags, int32_t K,
                                const int64_t *rho, const int64_t *beta, int64_t eps, int32_t permille,
                                int32_t move_thr, int32_t window, int64_t n_keys, const int64_t *off2,
                                int64_t n_req2, int32_t ahead2, int32_t interleave, int64_t *gs, int64_t *is,
                                int32_t *pr) {
    std::vector<TraceIn> ts{{off, n_req, group, contract, prefix, tick}};
    if (off2) ts.insert(ahead2 ? ts.begin() : ts.end(), {off2, n_req2, nullptr, nullptr, nullptr, nullptr});
    const Analysis A = analyse(keys, n_keys, ts, off2 && ahead2 ? 1 : 0, interleave);
    if (A.left) return 2;
    for (int64_t r = 0; r < n_req; ++r)
        if (contract[r] >= K) return 2;
    pcr::RunParams P{};
    P.C = (int32_t)C;
    P.G = G;
    P.K = K;
    P.flags = flags;
    int64_t sc = C * permille / 1000;
    if (sc < 1) sc = 1;
    P.s_cap = (int32_t)sc;
    P.g_cap = (int32_t)(C - sc);
    P.move_thr = move_thr;
    P.win = pcr::runs_windows(policy, (int32_t)C, window < 0);
    for (int32_t &n : P.win.n) n = window > 0 ? (policy == 1 || &n == P.win.n ? window : 0) : n;
    P.eps = eps;
    P.n_req = n_req;
    int64_t rmin = rho[0];
    for (int c = 0; c < K; ++c) rmin = rho[c] < rmin ? rho[c] : rmin;
    for (int c = 0; c < K; ++c) {
        P.rho[c] = rho[c];
        P.beta[c] = beta[c];
        P.invw[c] = (rmin << 16) / rho[c];
    }
    auto go = [&](auto pol) {
        constexpr int kPol = decltype(pol)::value;
        const bool ok = K == 1 ? replay_in<kPol, true>(A, P, n_prefix, gs, is, pr)
                               : replay_in<kPol, false>(A, P, n_prefix, gs, is, pr);
        return ok ? 0 : 1;
    };
    switch (policy) {
        case 0: return go(std::integral_constant<int, 0>());
        case 1: return go(std::integral_constant<int, 1>());
        case 2: return go(std::integral_constant<int, 2>());
        default: return go(std::integral_constant<int, 3>());
    }
}

// The rule that keeps an instance on runs (kPays*), what a batch makes of it,
// and which requests an instance is judged by.
extern "C" uint32_t runs_host_pays(int32_t policy, int32_t C, int32_t G, int64_t n_req, uint32_t n, uint32_t pieces,
                                   uint32_t blocks, uint32_t fresh, float load, float rounds) {
    return pcr::runs_pay(pcr::form_times(policy, C, policy == 3 ? C / G : C, n_req,
                                         pcr::RunsSample{n, pieces, blocks, fresh}), load, rounds);
}
extern "C" void runs_host_sample(const int64_t *req, int64_t n, uint32_t *sums) {
    uint64_t w = 0;
    for (int64_t i = 0; i < n; ++i) w += pcr::pack_sample((uint32_t)req[3 * i], (uint32_t)req[3 * i + 1], req[3 * i + 2]);
    const pcr::RunsSample s = pcr::unpack_sample(w);
    sums[0] = s.n, sums[1] = s.pieces, sums[2] = s.fresh, sums[3] = s.blocks;
}
extern "C" uint32_t runs_host_batch_pays(uint32_t pays, float runs_in, float general_in, float runs_all,
                                         float general_all) {
    return pcr::batch_pays(pays, runs_in, general_in, runs_all, general_all);
}
extern "C" int32_t runs_host_is_sampled(int64_t r, int64_t n_req) { return pcr::is_sampled(r, n_req); }
