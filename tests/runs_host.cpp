// runs_host.cpp -- the run-based replay (csrc/pc_runs.h) on the CPU: the
// wavefront is a structure of 64 lanes, LDS an array with bounds checks, and
// the trace analysis a plain map.  Built and driven by test_runs_cpu.py.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
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
PC_OP(+) PC_OP(-) PC_OP(&) PC_OP(|)
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
V<bool> operator!(const V<bool> &a) { return zip(a, a, [](bool x, bool) { return !x; }); }

uint32_t *g_lds;
int64_t g_lds_words;
[[noreturn]] void die(const char *what) {
    std::fprintf(stderr, "runs_host: %s\n", what);
    std::abort();
}
void check(const uint32_t *p) {
    if (p < g_lds || p >= g_lds + g_lds_words) die("LDS access out of range");
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
    static vl vmin(const vl &a, int64_t b) { return vmin(a, splat<int64_t>(b)); }
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
    static vu next_lane(const vu &a) {
        vu r;
        for (int i = 0; i < kLanes; ++i) r.v[i] = i + 1 < kLanes ? a.v[i + 1] : 0u;
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
    static uint64_t mulhi(uint64_t a, uint64_t b) { return (uint64_t)(((unsigned __int128)a * b) >> 64); }
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
    void st1(uint32_t *p, uint32_t at, uint32_t x) {
        check(p + at);
        p[at] = x;
    }
};
}  // namespace

#include "pc_runs.h"

namespace {

// Trace analysis on the host: ids, cuts, pieces (see pc_runs.h).
struct Analysis {
    std::vector<uint32_t> id;
    std::vector<uint8_t> weak;
    std::vector<pcr::RunReq> req;
    std::vector<pcr::RunPiece> piece;
};

Analysis analyse(const uint64_t *keys, const int64_t *off, const uint8_t *group, const uint8_t *contract,
                 const uint32_t *prefix, const int64_t *tick, int64_t n_req) {
    Analysis A;
    const int64_t n = n_req ? off[n_req] : 0;
    A.id.resize(n);
    A.weak.assign(n, 0);
    A.piece.resize(n);
    std::unordered_map<uint64_t, uint32_t> first;
    for (int64_t i = 0; i < n; ++i) A.id[i] = first.emplace(keys[i], (uint32_t)i).first->second;
    for (int64_t r = 0; r < n_req; ++r)
        for (int64_t i = off[r]; i < off[r + 1]; ++i)
            if (i == off[r] || A.id[i - 1] + 1 != A.id[i]) A.weak[A.id[i]] = 1;
    auto pieces = [&](int64_t r) {
        std::vector<std::pair<uint32_t, uint32_t>> p;    // id, depth
        for (int64_t i = off[r]; i < off[r + 1]; ++i)
            if (A.weak[A.id[i]]) p.push_back({A.id[i], (uint32_t)(i - off[r])});
        return p;
    };
    for (int64_t r = 0; r < n_req; ++r) {                // cuts where one of two equal starts ends
        const auto p = pieces(r);
        const uint32_t nf = (uint32_t)(off[r + 1] - off[r]);
        auto len = [&](size_t i) { return (i + 1 < p.size() ? p[i + 1].second : nf) - p[i].second; };
        for (size_t a = 0; a < p.size(); ++a)
            for (size_t b = 0; b < a; ++b)
                if (p[a].first == p[b].first && len(a) != len(b))
                    A.weak[p[a].first + (len(a) < len(b) ? len(a) : len(b))] = 1;
    }
    std::unordered_map<uint32_t, int> seen;
    for (int64_t r = 0; r < n_req; ++r) {
        const auto p = pieces(r);
        for (size_t a = 0; a < p.size(); ++a) {
            bool dup = false;
            for (size_t b = 0; b < a; ++b) dup = dup || p[a].first == p[b].first;
            A.piece[off[r] + a] = {p[a].first, p[a].second | (dup ? pcr::kPieceDup : 0u)};
        }
        const bool before = !seen.emplace(prefix[r], 1).second;
        A.req.push_back({(uint32_t)(off[r + 1] - off[r]), (uint32_t)p.size(),
                         group[r] | ((uint32_t)contract[r] << 8) | (before ? 1u << 16 : 0u), prefix[r],
                         tick ? tick[r] : r, (uint32_t)off[r], 0});
    }
    return A;
}

template <int kPol>
int replay(const Analysis &A, const pcr::RunParams &P, int64_t n_prefix, int64_t *gs, int64_t *is, int32_t *pr) {
    std::vector<uint32_t> lds(pcr::runs_lds_bytes(kPol, (int32_t)P.q) / 4, 0xDEADBEEFu);
    g_lds = lds.data();
    g_lds_words = (int64_t)lds.size();
    HostWave wv;
    pcr::RunReplay<HostWave, kPol> R(P, wv, lds.data());
    std::vector<uint8_t> adm(n_prefix + 1, 0);
    for (int64_t r = 0; r < P.n_req; ++r) {
        const pcr::RunReq &q = A.req[r];
        V<uint32_t> id = splat<uint32_t>(0), dep = splat<uint32_t>(0);
        for (uint32_t i = 0; i < q.np && i < 64; ++i) {
            id.v[i] = A.piece[q.ko + i].id;
            dep.v[i] = A.piece[q.ko + i].depth;
        }
        adm[q.prefix] = R.request((uint32_t)r, q, id, dep, adm[q.prefix] != 0);
        if (R.general) return 1;
        if (pr) {
            pr[4 * r] = R.last_h;
            pr[4 * r + 1] = R.last_m;
            pr[4 * r + 2] = R.last_e;
            pr[4 * r + 3] = R.last_o;
        }
    }
    const auto dend = R.raw_debt();
    for (int g = 0; g < P.G; ++g) {
        const int64_t probe = R.c_probe.v[g], hit = R.c_hit.v[g], dup = R.c_dup.v[g];
        const int64_t f[17] = {R.c_req.v[g], probe, hit, probe - hit, probe - hit - dup, R.evw.v[g], R.c_evc.v[g],
                               R.c_promo.v[g], R.c_gated.v[g], R.c_orph.v[g], dup, R.c_trunc.v[g],
                               P.n_req ? dend.v[g] : 0, R.d_max.v[g], R.d_sum.v[g], (int64_t)R.res.v[g],
                               (int64_t)R.res_max.v[g]};
        for (int k = 0; k < 17; ++k) gs[17 * g + k] = f[k];
    }
    const int64_t f[7] = {(int64_t)R.ev_total, (int64_t)R.s3_moves, (int64_t)R.s3_reins, (int64_t)R.s3_ghits,
                          (int64_t)R.s3_gins, R.resident, R.rmax};
    for (int k = 0; k < 7; ++k) is[k] = f[k];
    return 0;
}

}  // namespace

// The oracle's signature; `ring` overrides the ring size (0: the planner's).
// Returns 0, or 1 when the instance is left to the general kernel.
extern "C" int runs_host_replay(const uint64_t *keys, const int64_t *off, const uint8_t *group,
                                const uint8_t *contract, const uint32_t *prefix, const int64_t *tick, int64_t n_req,
                                int32_t G, int64_t n_prefix, int32_t policy, int64_t C, int32_t flags, int32_t K,
                                const int64_t *rho, const int64_t *beta, int64_t eps, int32_t permille,
                                int32_t move_thr, int32_t ring, int64_t *gs, int64_t *is, int32_t *pr) {
    const Analysis A = analyse(keys, off, group, contract, prefix, tick, n_req);
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
    P.q = (uint32_t)(ring ? ring : pcr::runs_ring((int32_t)C));
    P.eps = eps;
    P.n_req = n_req;
    int64_t rmin = rho[0];
    for (int c = 0; c < K; ++c) rmin = rho[c] < rmin ? rho[c] : rmin;
    for (int c = 0; c < K; ++c) {
        P.rho[c] = rho[c];
        P.beta[c] = beta[c];
        P.invw[c] = (rmin << 16) / rho[c];
    }
    switch (policy) {
        case 0: return replay<0>(A, P, n_prefix, gs, is, pr);
        case 1: return replay<1>(A, P, n_prefix, gs, is, pr);
        case 2: return replay<2>(A, P, n_prefix, gs, is, pr);
        default: return replay<3>(A, P, n_prefix, gs, is, pr);
    }
}
