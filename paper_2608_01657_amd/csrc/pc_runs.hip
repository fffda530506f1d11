// pc_runs.hip -- replay on runs of blocks (pc_runs.h) and the trace analysis
// that it needs, on gfx950.
//
// Analysis (per key buffer, shared by every instance that reads it):
//   runs_fill     clears the tables, bitmaps and flags
//   runs_insert   every key into an open-addressed table of positions (the
//                 least position of a key stays: its id); request starts
//                 and each prefix's first request
//   runs_link     ids of all positions; weak links
//   runs_list     per request: its pieces, duplicates among them, RunReq
//   runs_relist   the same again where duplicates added cuts (rare)
// Bound: runs_insert and runs_link make one random table access per key; the
// rest streams.
//
// Replay: one wavefront per instance, no barriers; bound by the chain of
// dependent instructions of a request.
#include "pc_internal.h"

#define PC_RUNS_FN __device__ __forceinline__
#include "pc_runs.h"

namespace pcr {
namespace {

#define DEV __device__ __forceinline__
#define GLOBAL __attribute__((address_space(1)))
#define CONST_AS __attribute__((address_space(4)))
#define LDS_AS __attribute__((address_space(3)))

// ------------------------------------------------------------ wavefront
struct DevWave {
    using vu = uint32_t;
    using vl = int64_t;
    using vb = bool;
    using Lds = LDS_AS uint32_t *;
    DEV vu lane() const { return (uint32_t)__lane_id(); }
    DEV vu vu0(uint32_t x) const { return x; }
    DEV vl vl0(int64_t x) const { return x; }
    // LDS operations of a wavefront execute in order; the fence keeps the
    // compiler from moving a lane's load above another lane's store
    DEV static void sync() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
    }
    DEV static uint64_t ballot(bool b) { return __ballot(b); }
    DEV static bool of_mask(uint64_t m) { return (m >> __lane_id()) & 1ull; }
    DEV static int popc(uint64_t m) { return __popcll(m); }
    DEV static int ffs(uint64_t m) { return __builtin_ctzll(m); }      // m != 0
    DEV static int clz(uint64_t m) { return __builtin_clzll(m); }      // m != 0
    DEV static uint32_t rfl(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
    DEV static uint32_t rdl(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }
    DEV static int64_t rdl64(int64_t v, int l) {
        const uint32_t lo = rdl((uint32_t)(uint64_t)v, l), hi = rdl((uint32_t)((uint64_t)v >> 32), l);
        return (int64_t)(((uint64_t)hi << 32) | lo);
    }
    template <class T>
    DEV static T sel(bool m, T a, T b) { return m ? a : b; }
    template <class T>
    DEV static T vmin(T a, T b) { return a < b ? a : b; }
    template <class T>
    DEV static T vmax(T a, T b) { return a > b ? a : b; }
    // DPP steps: within each row of 16 lanes, then across rows (row_bcast:15
    // into rows 1 and 3, row_bcast:31 into rows 2 and 3)
    template <int kCtrl, int kRowMask>
    DEV static uint32_t dpp(uint32_t old, uint32_t v) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, kCtrl, kRowMask, 0xF, false);
    }
    template <int kCtrl, int kRowMask>
    DEV static int64_t dpp64(int64_t v) {
        const uint32_t lo = dpp<kCtrl, kRowMask>((uint32_t)(uint64_t)v, (uint32_t)(uint64_t)v);
        const uint32_t hi = dpp<kCtrl, kRowMask>((uint32_t)((uint64_t)v >> 32), (uint32_t)((uint64_t)v >> 32));
        return (int64_t)(((uint64_t)hi << 32) | lo);
    }
    DEV static uint32_t scan(uint32_t v) {
        v += dpp<0x111, 0xF>(0u, v);
        v += dpp<0x112, 0xF>(0u, v);
        v += dpp<0x114, 0xF>(0u, v);
        v += dpp<0x118, 0xF>(0u, v);
        v += dpp<0x142, 0xA>(0u, v);
        v += dpp<0x143, 0xC>(0u, v);
        return v;
    }
    DEV static uint32_t wsum(uint32_t v) { return rdl(scan(v), 63); }
    DEV static uint32_t wmax(uint32_t v) {
        v = vmax(v, dpp<0x111, 0xF>(0u, v));
        v = vmax(v, dpp<0x112, 0xF>(0u, v));
        v = vmax(v, dpp<0x114, 0xF>(0u, v));
        v = vmax(v, dpp<0x118, 0xF>(0u, v));
        v = vmax(v, dpp<0x142, 0xA>(0u, v));
        v = vmax(v, dpp<0x143, 0xC>(0u, v));
        return rdl(v, 63);
    }
    DEV static int64_t wmax64(int64_t v) {     // a lane without a source lane keeps its own value
        v = vmax(v, dpp64<0x111, 0xF>(v));
        v = vmax(v, dpp64<0x112, 0xF>(v));
        v = vmax(v, dpp64<0x114, 0xF>(v));
        v = vmax(v, dpp64<0x118, 0xF>(v));
        v = vmax(v, dpp64<0x142, 0xA>(v));
        v = vmax(v, dpp64<0x143, 0xC>(v));
        return rdl64(v, 63);
    }
    DEV static uint32_t mbcnt(uint64_t m) {
        return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    }
    DEV static uint32_t next_lane(uint32_t v) {    // lane i: the value of lane i + 1
        return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(((uint32_t)__lane_id() + 1u) << 2), (int)v);
    }
    DEV static int64_t widen(uint32_t v) { return (int64_t)(uint64_t)v; }
    DEV static int64_t mul_shr16(int64_t a, int64_t w) {      // a, w >= 0 in the lanes that use it
        const uint64_t x = (uint64_t)a, y = (uint64_t)w;
        return (int64_t)((__umul64hi(x, y) << 48) | ((x * y) >> 16));
    }
    DEV static uint64_t mulhi(uint64_t a, uint64_t b) { return __umul64hi(a, b); }
    DEV static uint64_t udiv(uint64_t a, uint64_t b) { return a / b; }
    DEV static uint32_t ld(Lds p, uint32_t at) { return p[at]; }
    DEV static void st(bool m, Lds p, uint32_t at, uint32_t x) {
        if (m) p[at] = x;
    }
    DEV void st1(Lds p, uint32_t at, uint32_t x) {
        if (__lane_id() == 0) p[at] = x;
    }
};

// ------------------------------------------------------------ analysis
constexpr int kT = 256;
// A key that has not found its place after this many steps ends the attempt
// (its traces are left to the general kernel): at load 1/2 only keys made to
// collide get there.
constexpr uint32_t kMaxProbe = 2048;
constexpr uint32_t kResolved = 0x80000000u;    // id[pos] holds the id, not yet the table slot

__global__ __launch_bounds__(kT) void runs_fill(uint4 *ones, int64_t n_ones, uint4 *zeros, int64_t n_zeros) {
    const int64_t i0 = (int64_t)blockIdx.x * kT + threadIdx.x, step = (int64_t)gridDim.x * kT;
    for (int64_t i = i0; i < n_ones; i += step) ones[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    for (int64_t i = i0; i < n_zeros; i += step) zeros[i] = make_uint4(0u, 0u, 0u, 0u);
}

DEV uint32_t key_slot(uint64_t k, uint32_t slots) {
    k ^= k >> 32;
    k *= 0x9E3779B97F4A7C15ull;
    k ^= k >> 29;
    k *= 0xBF58476D1CE4E5B9ull;
    return __umulhi((uint32_t)(k >> 32), slots);
}

// the last entry of a[0..n) whose `blk0` is at or below b (a[0].blk0 <= b)
template <class T>
DEV int32_t find_block(const T *a, int32_t n, uint32_t b, uint32_t T::*blk0) {
    int32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (a[mid].*blk0 <= b) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Request r of a trace: false if the general kernel would refuse it (the
// contract aside, which depends on the instance).
DEV bool request_ok(const DevTrace &T, int64_t r, int64_t &ko, int64_t &nf) {
    ko = T.key_off[r];
    nf = T.key_off[r + 1] - ko;
    const int64_t t = T.tick ? T.tick[r] : r;
    const int64_t tp = T.tick && r > 0 ? T.tick[r - 1] : 0;
    return !(T.group[r] >= T.n_groups || (int64_t)T.prefix[r] >= T.n_prefix || ko < 0 || nf < 0 ||
             ko + nf > T.n_keys || nf > T.max_req_blocks || t < 0 || t < tp);
}

// Blocks [0, nb_pos): positions of the key buffers; then requests.
__global__ __launch_bounds__(kT) void runs_insert(RunsArgs A) {
    if (blockIdx.x >= A.nb_pos) {
        const uint32_t b = blockIdx.x - A.nb_pos;
        const int32_t ti = find_block(A.traces, A.n_traces, b, &DevRunTrace::blk0);
        const DevRunTrace &R = A.traces[ti];
        const DevTrace &T = A.tr[R.trace];
        const int64_t r = (int64_t)(b - R.blk0) * kT + threadIdx.x;
        if (r >= T.n_req) return;
        int64_t ko, nf;
        if (!request_ok(T, r, ko, nf)) {
            A.tflag[ti] = 1;
            return;
        }
        if (nf > 0) atomicOr(A.start + A.bufs[R.buf].bits0 + (ko >> 5), 1u << (ko & 31));
        atomicMin(A.first + R.first0 + T.prefix[r], (uint32_t)r);
        return;
    }
    const int32_t bi = find_block(A.bufs, A.n_bufs, blockIdx.x, &DevKeyBuf::blk0);
    const DevKeyBuf &B = A.bufs[bi];
    const int64_t pos = (int64_t)(blockIdx.x - B.blk0) * kT + threadIdx.x;
    if (pos >= B.n) return;
    const GLOBAL uint64_t *keys = (const GLOBAL uint64_t *)B.keys;
    uint32_t *tab = A.table + B.tab0;
    const uint64_t k = keys[pos];
    uint32_t at = key_slot(k, B.slots);
    for (uint32_t it = 0; it < kMaxProbe; ++it) {
        uint32_t v = tab[at];
        if (v == kEmpty) v = atomicCAS(tab + at, kEmpty, (uint32_t)pos);
        if (v == kEmpty) break;
        if (keys[v] == k) {
            if ((uint32_t)pos < v) atomicMin(tab + at, (uint32_t)pos);
            break;
        }
        at = at + 1u == B.slots ? 0u : at + 1u;
        if (it + 1 == kMaxProbe) A.bflag[2 * bi] = 1;
    }
    A.id[B.id0 + pos] = at;
}

__global__ __launch_bounds__(kT) void runs_link(RunsArgs A) {
    const int32_t bi = find_block(A.bufs, A.n_bufs, blockIdx.x, &DevKeyBuf::blk0);
    const DevKeyBuf &B = A.bufs[bi];
    if (A.bflag[2 * bi]) return;      // (its slots may be wrong)
    const int64_t pos = (int64_t)(blockIdx.x - B.blk0) * kT + threadIdx.x;
    const uint32_t *tab = A.table + B.tab0;
    uint32_t *id = A.id + B.id0;
    uint32_t x = 0;
    const bool in = pos < B.n;
    if (in) x = tab[id[pos]];
    // the id before it: the lane before, or for lane 0 from memory, where
    // another wavefront may have replaced the slot by the id already
    uint32_t before = (uint32_t)__shfl_up((int)x, 1);
    if ((threadIdx.x & 63) == 0 && in && pos > 0) {
        const uint32_t s = __hip_atomic_load(id + pos - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        before = (s & kResolved) ? s & ~kResolved : tab[s];
    }
    if (!in) return;
    __hip_atomic_store(id + pos, x | kResolved, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool st = (A.start[B.bits0 + (pos >> 5)] >> (pos & 31)) & 1u;
    if (pos == 0 || st || before + 1u != x) atomicOr(A.weak + B.bits0 + (x >> 5), 1u << (x & 31));
}

// One wavefront per request.  kAgain: only where a first pass added cuts.
template <bool kAgain>
__global__ __launch_bounds__(kT) void runs_list(RunsArgs A) {
    __shared__ uint32_t s_id[kT / 64][64], s_dep[kT / 64][64];
    const int32_t ti = find_block(A.traces, A.n_traces, blockIdx.x, &DevRunTrace::blk1);
    const DevRunTrace &R = A.traces[ti];
    const DevKeyBuf &B = A.bufs[R.buf];
    if (kAgain && A.bflag[2 * R.buf + 1] == 0) return;
    if (A.tflag[ti] || A.bflag[2 * R.buf]) return;
    const DevTrace &T = A.tr[R.trace];
    const int w = (int)threadIdx.x >> 6;
    const uint32_t lane = threadIdx.x & 63;
    const int64_t r = (int64_t)(blockIdx.x - R.blk1) * (kT / 64) + __builtin_amdgcn_readfirstlane(w);
    if (r >= T.n_req) return;
    int64_t ko, nf;
    request_ok(T, r, ko, nf);          // (valid: the flag above is clear)
    const uint32_t *id = A.id + B.id0;
    const uint32_t *weak = A.weak + B.bits0;
    uint32_t np = 0;
    for (int64_t j0 = 0; j0 < nf; j0 += 64) {
        const int64_t j = j0 + lane;
        uint32_t x = 0;
        bool cut = false;
        if (j < nf) {
            x = id[ko + j] & ~kResolved;
            cut = (weak[x >> 5] >> (x & 31)) & 1u;
        }
        const uint64_t m = __ballot(cut);
        const uint32_t k = np + DevWave::mbcnt(m);
        if (cut && k < 64u) {
            s_id[w][k] = x;
            s_dep[w][k] = (uint32_t)j;
        }
        np += (uint32_t)__popcll(m);
    }
    DevWave::sync();
    uint32_t pid = 0, dep = 0;
    if (np <= 64u) {
        const bool in = lane < np;
        if (in) { pid = s_id[w][lane]; dep = s_dep[w][lane]; }
        bool dup = false;
        if (np > 1u) {
            const uint32_t nx = DevWave::next_lane(dep);
            const uint32_t len = (lane + 1u < np ? nx : (uint32_t)nf) - dep;
            for (uint32_t i = 0; i + 1 < np; ++i) {
                const uint32_t a = DevWave::rdl(pid, (int)i), la = DevWave::rdl(len, (int)i);
                const bool same = in && lane > i && pid == a;
                dup = dup || same;
                if (!kAgain && same && len != la) {     // cut where the shorter of the two ends
                    const uint32_t c = a + (len < la ? len : la);
                    atomicOr(A.weak + B.bits0 + (c >> 5), 1u << (c & 31));
                    A.bflag[2 * R.buf + 1] = 1;
                }
            }
        }
        // the pieces are kept at the request's own key positions; another
        // trace's request may start among them when traces overlap
        const bool clash = in && lane > 0 && ((A.start[B.bits0 + ((ko + lane) >> 5)] >> ((ko + lane) & 31)) & 1u);
        if (__ballot(clash)) {
            if (lane == 0) A.tflag[ti] = 1;
            return;
        }
        if (in) {
            RunPiece p;
            p.id = pid;
            p.depth = dep | (dup ? kPieceDup : 0u);
            ((RunPiece *)(A.table + B.tab0))[ko + lane] = p;
        }
    }
    if (lane == 0) {
        RunReq q;
        q.n_full = (uint32_t)nf;
        q.np = np;
        q.prefix = T.prefix[r];
        q.info = (uint32_t)T.group[r] | ((uint32_t)T.contract[r] << 8) |
                 (A.first[R.first0 + q.prefix] < (uint32_t)r ? 1u << 16 : 0u);
        q.tick = T.tick ? T.tick[r] : r;
        q.ko = (uint32_t)ko;
        q.pad = 0;
        A.req[R.req0 + r] = q;
    }
}

// ------------------------------------------------------------ replay
DEV RunReq load_req(const CONST_AS RunReq *req, int64_t r) {
    RunReq q;
    q.n_full = req[r].n_full;
    q.np = req[r].np;
    q.info = req[r].info;
    q.prefix = req[r].prefix;
    q.tick = req[r].tick;
    q.ko = req[r].ko;
    return q;
}

template <int kPol>
DEV void replay_runs(const RunsArgs &A, const DevInst &I, const DevTrace &T, const DevRunTrace &R, int id, uint8_t *ws,
                     int64_t *stats, int32_t *per_req, LDS_AS uint32_t *lds) {
    RunParams P;
    P.C = I.capacity;
    P.G = T.n_groups;
    P.K = I.n_contracts;
    P.flags = I.flags;
    P.s_cap = I.s_cap;
    P.g_cap = I.g_cap;
    P.move_thr = I.move_thr;
    P.q = (uint32_t)I.run_ring;
    P.eps = I.eps;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        P.rho[c] = I.rho[c];
        P.beta[c] = I.beta[c];
        P.invw[c] = I.invw[c];
    }
    P.n_req = T.n_req;
    const uint32_t lane = (uint32_t)__lane_id();
    GLOBAL uint32_t *bits = (GLOBAL uint32_t *)(ws + I.ws_bits);
    if (kPol == 2) {
        for (int i = (int)lane; i < I.n_prefix_words; i += 64) bits[i] = 0u;
        __threadfence();
    }
    const DevKeyBuf &B = A.bufs[R.buf];
    const CONST_AS RunReq *req = (const CONST_AS RunReq *)(uintptr_t)(A.req + R.req0);
    const GLOBAL uint2 *piece = (const GLOBAL uint2 *)(A.table + B.tab0);
    int32_t *pr = (per_req && I.per_req_off >= 0) ? per_req + I.per_req_off : nullptr;
    DevWave wv;
    RunReplay<DevWave, kPol> X(P, wv, lds);
    const int64_t n = P.n_req;
    // request r runs while r + 1's pieces and prefix bit and r + 2's
    // descriptor are on their way
    RunReq q = {}, nx = {};
    uint2 pc = make_uint2(0u, 0u);
    uint32_t word = 0;           // (lane 0) admitted bits around q.prefix
    if (n > 0) {
        q = load_req(req, 0);
        if (n > 1) nx = load_req(req, 1);
        if (lane < q.np && q.np <= 64u) pc = make_uint2(piece[q.ko + lane].x, piece[q.ko + lane].y);
    }
    for (int64_t r = 0; r < n; ++r) {
        uint2 pn = make_uint2(0u, 0u);
        uint32_t wn = 0;
        RunReq nn = {};
        if (r + 1 < n) {
            if (lane < nx.np && nx.np <= 64u) pn = make_uint2(piece[nx.ko + lane].x, piece[nx.ko + lane].y);
            if (kPol == 2 && lane == 0) wn = bits[nx.prefix >> 5];
            if (r + 2 < n) nn = load_req(req, r + 2);
        }
        bool adm = false;
        if (kPol == 2) adm = (DevWave::rfl(word) >> (q.prefix & 31)) & 1u;
        const bool now = X.request((uint32_t)r, q, pc.x, pc.y, adm);
        if (X.general) return;       // the general kernel replays the instance
        if (kPol == 2 && now && !adm) {
            word |= 1u << (q.prefix & 31);
            if (lane == 0) bits[q.prefix >> 5] = word;
        }
        if (kPol == 2 && (nx.prefix >> 5) == (q.prefix >> 5)) wn = word;
        if (pr && lane == 0) {
            int32_t *o = pr + 4 * r;
            o[0] = X.last_h;
            o[1] = X.last_m;
            o[2] = X.last_e;
            o[3] = X.last_o;
        }
        q = nx;
        nx = nn;
        pc = pn;
        word = wn;
    }
    // stats record: 64 groups x 17 int64, then the instance block
    int64_t *st = stats + (int64_t)id * kRecordWords;
    int64_t *o = st + lane * kGroupFields;
    const bool grp = (int)lane < P.G;
    const int64_t v[kGroupFields] = {X.c_req, X.c_probe, X.c_hit, X.c_probe - X.c_hit, X.c_probe - X.c_hit - X.c_dup,
                                     X.evw, X.c_evc, X.c_promo, X.c_gated, X.c_orph, X.c_dup, X.c_trunc,
                                     n > 0 ? X.raw_debt() : 0, X.d_max, X.d_sum, (int64_t)X.res, (int64_t)X.res_max};
#pragma unroll
    for (int f = 0; f < kGroupFields; ++f) o[f] = grp ? v[f] : 0;
    if (lane == 0) {
        int64_t *qq = st + kInstOffset;
        qq[0] = (int64_t)X.ev_total;
        qq[1] = (int64_t)X.s3_moves;
        qq[2] = (int64_t)X.s3_reins;
        qq[3] = (int64_t)X.s3_ghits;
        qq[4] = (int64_t)X.s3_gins;
        qq[5] = (int64_t)X.resident;
        qq[6] = (int64_t)X.rmax;
        qq[7] = 0;
        A.done[id] = 1;
    }
}

__global__ __launch_bounds__(64) void runs_replay(RunsArgs A, const int32_t *__restrict__ order, uint8_t *ws,
                                                  int64_t *stats, int32_t *per_req) {
    extern __shared__ __align__(16) uint32_t runs_smem[];
    const int id = order[blockIdx.x];
    const DevInst &I = A.inst[id];
    const DevRunTrace &R = A.traces[I.run_trace];
    if (A.tflag[I.run_trace] || A.bflag[2 * R.buf]) return;
    const DevTrace &T = A.tr[I.trace];
    LDS_AS uint32_t *lds = (LDS_AS uint32_t *)runs_smem;
    if (I.policy == kLRU) replay_runs<kLRU>(A, I, T, R, id, ws, stats, per_req, lds);
    else if (I.policy == kS3) replay_runs<kS3>(A, I, T, R, id, ws, stats, per_req, lds);
    else if (I.policy == kSQ) replay_runs<kSQ>(A, I, T, R, id, ws, stats, per_req, lds);
    else replay_runs<kPS>(A, I, T, R, id, ws, stats, per_req, lds);
}

}  // namespace

hipError_t launch_runs_analysis(const RunsArgs &A, uint4 *ones, int64_t n_ones, uint4 *zeros, int64_t n_zeros,
                                uint32_t nb_req, uint32_t nb_list, hipStream_t s) {
    const int64_t nb = (n_ones + n_zeros + 4 * kT - 1) / (4 * kT);
    hipLaunchKernelGGL(runs_fill, dim3((unsigned)(nb < 8192 ? (nb > 0 ? nb : 1) : 8192)), dim3(kT), 0, s, ones, n_ones,
                       zeros, n_zeros);
    hipLaunchKernelGGL(runs_insert, dim3(A.nb_pos + nb_req), dim3(kT), 0, s, A);
    if (A.nb_pos > 0) hipLaunchKernelGGL(runs_link, dim3(A.nb_pos), dim3(kT), 0, s, A);
    hipLaunchKernelGGL(runs_list<false>, dim3(nb_list), dim3(kT), 0, s, A);
    hipLaunchKernelGGL(runs_list<true>, dim3(nb_list), dim3(kT), 0, s, A);
    return hipGetLastError();
}

hipError_t runs_set_lds_limit(int32_t lds_bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&runs_replay),
                               hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
}

hipError_t launch_runs_replay(const RunsArgs &A, const int32_t *d_order, int32_t n_launch, int32_t lds_bytes,
                              uint8_t *ws, int64_t *stats, int32_t *per_req, hipStream_t s) {
    hipLaunchKernelGGL(runs_replay, dim3((unsigned)n_launch), dim3(64), (size_t)lds_bytes, s, A, d_order, ws, stats,
                       per_req);
    return hipGetLastError();
}

}  // namespace pcr
