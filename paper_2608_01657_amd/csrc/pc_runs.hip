// pc_runs.hip -- replay on runs of blocks (pc_runs.h) and the trace analysis
// that it needs, on gfx950.
//
// Analysis (per key buffer, shared by every instance that reads it):
//   runs_fill     clears the tables, bitmaps and flags
//   runs_insert   every key into an open-addressed table of positions (the
//                 least position of a key stays: its id); request starts
//                 and each prefix's first request
//   runs_link     ids of all positions; weak links
//   runs_list     per request: its pieces, duplicates among them, RunReq, and
//                 sums over a sample of the requests
//   runs_list     again (kAgain) for key buffers where duplicates added cuts;
//                 the form that each instance takes
// Bound: runs_insert and runs_link make one random table access per key; the
// rest streams.  16 one-touch traces of 50,000 requests (119 M keys): insert
// 5.0 ms, link 2.0, list 0.6, fill 0.15; 64 traces of conversations, 100,000
// requests each (648 M keys): insert 32.7, link 9.7, list 4.9, fill 1.3.
//
// Replay: one wavefront per instance, no barriers; bound by the chain of
// dependent instructions of a request, whatever its number of blocks.  1,024
// one-touch instances of 4,096 blocks, 50,000 requests each: 117 ms with keys
// and analysis, 2.1 to 2.3 us a request; the general kernels, a workgroup of
// four wavefronts and a step per 256 blocks, take 939 ms (two instances to a
// CU, 18.8 us a request).
#include "pc.h"
#include "pc_internal.h"

#define PC_RUNS_FN __device__ __forceinline__
#include "pc_runs.h"

namespace pcr {
namespace {

#define DEV __device__ __forceinline__
#define GLOBAL __attribute__((address_space(1)))
#define LDS_AS __attribute__((address_space(3)))

// ------------------------------------------------------------ wavefront
// (LLVM's intrinsic; clang has no builtin for it)
extern "C" __device__ uint32_t pc_writelane(uint32_t x, uint32_t l, uint32_t v) __asm("llvm.amdgcn.writelane.i32");
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
    // (upper words first, then the lower words of those that have the most:
    // half the instructions of six steps on 64-bit values)
    DEV static int64_t wmax64(int64_t v) {
        const int32_t hi = (int32_t)(v >> 32);
        int32_t h = hi;
        h = vmax(h, (int32_t)dpp<0x111, 0xF>(0x80000000u, (uint32_t)h));
        h = vmax(h, (int32_t)dpp<0x112, 0xF>(0x80000000u, (uint32_t)h));
        h = vmax(h, (int32_t)dpp<0x114, 0xF>(0x80000000u, (uint32_t)h));
        h = vmax(h, (int32_t)dpp<0x118, 0xF>(0x80000000u, (uint32_t)h));
        h = vmax(h, (int32_t)dpp<0x142, 0xA>(0x80000000u, (uint32_t)h));
        h = vmax(h, (int32_t)dpp<0x143, 0xC>(0x80000000u, (uint32_t)h));
        const int32_t top = (int32_t)rdl((uint32_t)h, 63);
        const uint32_t lo = wmax(hi == top ? (uint32_t)(uint64_t)v : 0u);
        return (int64_t)(((uint64_t)(uint32_t)top << 32) | lo);
    }
    DEV static uint32_t mbcnt(uint64_t m) {
        return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    }
    DEV static uint32_t setlane(uint32_t v, int l, uint32_t x) {
        return pc_writelane(x, (uint32_t)l, v);
    }
    DEV static void st_all(Lds p, uint32_t at, uint32_t x) { p[at] = x; }
    DEV static uint32_t next_lane(uint32_t v) {    // lane i: the value of lane i + 1
        return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(((uint32_t)__lane_id() + 1u) << 2), (int)v);
    }
    // device memory, lanes m; gor_bit: one bit of a bitmap
    DEV static uint32_t gld(bool m, const uint32_t *p, uint32_t at) { return m ? p[at] : 0u; }
    DEV static void gst2(bool m, uint32_t *p, uint32_t at, uint32_t x, uint32_t y) {
        if (m) ((uint2 *)p)[at] = make_uint2(x, y);
    }
    DEV static void gor_bit(bool m, uint32_t *p, uint32_t i) {
        if (m) atomicOr(p + (i >> 5), 1u << (i & 31));
    }
    DEV static bool bit(uint32_t w, uint32_t i) { return (w >> (i & 31)) & 1u; }
    DEV static int64_t widen(uint32_t v) { return (int64_t)(uint64_t)v; }
    DEV static int64_t mul_shr16(int64_t a, int64_t w) {      // a, w >= 0 in the lanes that use it
        const uint64_t x = (uint64_t)a, y = (uint64_t)w;
        return (int64_t)((__umul64hi(x, y) << 48) | ((x * y) >> 16));
    }
    DEV static int64_t mul_sat62(int64_t a, uint32_t b) {     // min(a b, 2^62) for a below 2^41
        const uint64_t lo = (uint64_t)a * b;
        return __umul64hi((uint64_t)a, b) != 0 || lo > (1ull << 62) ? (int64_t)1 << 62 : (int64_t)lo;
    }
    // keep a uniform value in a vector register; and back
    template <class T>
    DEV static T hold(T x) {
        asm volatile("" : "+v"(x));
        return x;
    }
    DEV static uint32_t uni(uint32_t v) { return rfl(v); }
    DEV static uint64_t udiv(uint64_t a, uint64_t b) { return a / b; }
    DEV static uint32_t ld(Lds p, uint32_t at) { return p[at]; }
    DEV static void st(bool m, Lds p, uint32_t at, uint32_t x) {
        if (m) p[at] = x;
    }
    DEV static uint32_t ld_if(bool m, Lds p, uint32_t at) { return m ? p[at] : 0u; }
    DEV uint32_t ld1(Lds p, uint32_t at) const { return rfl(p[at]); }
    // one word by lane 0; the others write a word of their own in scratch,
    // so that no branch or execution mask is needed
    template <int N>
    DEV void st1(Lds p, uint32_t at, Lds scratch, uint32_t x, uint32_t y, uint32_t z) const {
        const Lds to = __lane_id() == 0 ? p + at : scratch + __lane_id();
        to[0] = x;
        to[64] = y;
        if (N > 2) to[128] = z;
    }
    DEV static uint32_t mad01(uint32_t a, uint32_t b, uint32_t c) { return (a ? b : 0u) + c; }      // a is 0 or 1
    // a uniform value that stays in a scalar register
    DEV static uint32_t keep(uint32_t x) { return rfl(x); }
    DEV static int64_t mad64(uint32_t a, int32_t b, int64_t c) { return (int64_t)(int32_t)a * (int64_t)b + c; }
    DEV static bool likely(bool x) { return __builtin_expect(x, true); }
    DEV static bool unlikely(bool x) { return __builtin_expect(x, false); }
};

// ------------------------------------------------------------ analysis
constexpr int kT = 256;
// A key that has not found its place after this many steps ends the attempt
// (its traces are left to the general kernel): at load 1/2 only keys made to
// collide get there.
constexpr uint32_t kMaxProbe = 2048;

__global__ __launch_bounds__(kT) void runs_fill(uint4 *ones, int64_t n_ones, uint4 *zeros, int64_t n_zeros) {
    const int64_t i0 = (int64_t)blockIdx.x * kT + threadIdx.x, step = (int64_t)gridDim.x * kT;
    for (int64_t i = i0; i < n_ones; i += step) ones[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    for (int64_t i = i0; i < n_zeros; i += step) zeros[i] = make_uint4(0u, 0u, 0u, 0u);
}

// (multipliers: 2^64 over the golden ratio, and splitmix64's first)
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
// contract aside, which depends on the instance), or if its tick is 2^32 or
// more behind the one before it.
DEV bool request_ok(const DevTrace &T, int64_t r, int64_t &ko, int64_t &nf) {
    ko = T.key_off[r];
    nf = T.key_off[r + 1] - ko;
    const int64_t t = T.tick ? T.tick[r] : r;
    const int64_t tp = T.tick && r > 0 ? T.tick[r - 1] : 0;
    return !(T.group[r] >= T.n_groups || (int64_t)T.prefix[r] >= T.n_prefix || ko < 0 || nf < 0 ||
             ko + nf > T.n_keys || nf > T.max_req_blocks || t < 0 || t < tp || t - tp > (int64_t)0xFFFFFFFF);
}

// The keys of a buffer that are analysed: [base, base + n) of it.  Positions
// and ids count from base on.
struct Span {
    int64_t base, n;
};
DEV Span span_of(const RunsArgs &A, const DevKeyBuf &B) {
    if (B.trace < 0) return {0, B.n};
    const DevTrace &T = A.tr[B.trace];
    const int64_t a = T.key_off[0], e = T.key_off[T.n_req];
    // (else some request is malformed, and the trace is left)
    const bool ok = a >= 0 && e >= a && e <= T.n_keys && e - a <= B.n;
    return {a, ok ? e - a : 0};
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
        const DevKeyBuf &B = A.bufs[R.buf];
        const Span S = span_of(A, B);
        int64_t ko, nf;
        if (!request_ok(T, r, ko, nf) || ko < S.base || ko - S.base + nf > S.n) {
            A.tflag[ti] = 1;
            return;
        }
        uint32_t *marks = A.start + B.bits0;
        const int32_t c = T.contract[r];
        if (c > A.cmax[ti]) atomicMax(A.cmax + ti, c);
        request_marks(ko - S.base, nf, r + 1 == T.n_req, S.n,
                      [&](int64_t at) { atomicOr(marks + (at >> 5), 1u << (at & 31)); });
        atomicMin(A.first + R.first0 + T.prefix[r], (uint32_t)r);
        return;
    }
    const int32_t bi = find_block(A.bufs, A.n_bufs, blockIdx.x, &DevKeyBuf::blk0);
    const DevKeyBuf &B = A.bufs[bi];
    const Span S = span_of(A, B);
    const int64_t pos = (int64_t)(blockIdx.x - B.blk0) * kT + threadIdx.x;
    if (pos >= S.n) return;
    const GLOBAL uint64_t *keys = (const GLOBAL uint64_t *)B.keys + S.base;
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
    const bool in = pos < span_of(A, B).n;
    if (in) x = tab[id[pos]];
    // the id before it: the lane before, or for lane 0 from memory, where
    // another wavefront may have replaced the slot by the id already
    uint32_t before = (uint32_t)__shfl_up((int)x, 1);
    if ((threadIdx.x & 63) == 0 && in && pos > 0) {
        const uint32_t s = __hip_atomic_load(id + pos - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        before = (s & kRunsResolved) ? s & ~kRunsResolved : tab[s];
    }
    if (!in) return;
    __hip_atomic_store(id + pos, x | kRunsResolved, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool st = (A.start[B.bits0 + (pos >> 5)] >> (pos & 31)) & 1u;
    if (pos == 0 || st || before + 1u != x) atomicOr(A.weak + B.bits0 + (x >> 5), 1u << (x & 31));
}

// Which form each instance takes, by one workgroup.
DEV void choose_form(const RunsArgs &A) {
    // longest: on runs of those that pay, of all that can; in the general
    // kernels of the rest, of those that can not, of all
    // (words of positive floats sort as the floats do)
    __shared__ uint32_t s_most[kT / 64][6];
    uint32_t m[6] = {};                  // m[5]: how many are left
    auto times = [&](const DevInst &I, const DevTrace &T) {
        return form_times(I.policy, I.capacity, I.policy == kSQ ? I.capacity / T.n_groups : I.capacity, T.n_req,
                          unpack_sample(A.sample[kSampleStride * I.run_trace]));
    };
    FormTimes own{};      // of the thread's first instance
    const float rounds = (float)((A.n_run + A.n_cu - 1) / A.n_cu);
    for (int32_t i = (int32_t)threadIdx.x; i < A.n_inst; i += kT) {
        const DevInst &I = A.inst[i];
        if (I.run_trace < 0) continue;
        const DevTrace &T = A.tr[I.trace];
        const FormTimes t = times(I, T);
        if (i < kT) own = t;
        const uint32_t r = __float_as_uint((float)T.n_req * t.first), g = __float_as_uint((float)T.n_req * t.general);
        const bool can = !A.tflag[I.run_trace] && !A.bflag[2 * A.traces[I.run_trace].buf] &&
                         A.cmax[I.run_trace] < I.n_contracts;
        const bool in = can && (runs_pay(t, A.load, rounds) & kPaysFirst);
        m[0] = DevWave::vmax(m[0], in ? r : 0u);
        m[1] = DevWave::vmax(m[1], can ? r : 0u);
        m[2] = DevWave::vmax(m[2], in ? 0u : g);
        m[3] = DevWave::vmax(m[3], can ? 0u : g);
        m[4] = DevWave::vmax(m[4], g);
        m[5] += in ? 0u : 1u;
    }
    const int w = (int)threadIdx.x >> 6;
    for (int k = 0; k < 6; ++k) {
        const uint32_t x = k < 5 ? DevWave::wmax(m[k]) : DevWave::wsum(m[k]);
        if ((threadIdx.x & 63) == 0) s_most[w][k] = x;
    }
    __syncthreads();
    float most[5] = {};
    uint32_t left = 0;
    for (int q = 0; q < kT / 64; ++q) {
        for (int k = 0; k < 5; ++k) most[k] = DevWave::vmax(most[k], __uint_as_float(s_most[q][k]));
        left += s_most[q][5];
    }
    const float part = A.load * (float)left / (float)A.n_run, load = part > 1.0f ? part : 1.0f;    // of those left
    for (int32_t i = (int32_t)threadIdx.x; i < A.n_inst; i += kT) {
        const DevInst &I = A.inst[i];
        if (I.run_trace >= 0)
            A.pays[i] = batch_pays(runs_pay(i < kT ? own : times(I, A.tr[I.trace]), A.load, rounds), most[0],
                                   most[2] * load, most[1] + most[3] * load, most[4] * A.load);
    }
}

// One wavefront per request.  kAgain: only where a first pass added cuts.
template <bool kAgain>
__global__ __launch_bounds__(kT) void runs_list(RunsArgs A) {
    __shared__ uint32_t s_list[kT / 64][128];
    if (kAgain && blockIdx.x == 0) choose_form(A);      // (the first pass has sampled every trace)
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
    ko -= span_of(A, B).base;
    RunsBuf V;
    V.id = A.id + B.id0;
    V.weak = A.weak + B.bits0;
    V.cuts = A.cuts + B.bits0;
    V.start = A.start + B.bits0;
    V.piece = A.table + B.tab0;
    DevWave wv;
    const RunsListed L = list_request<DevWave, kAgain>(wv, V, (uint32_t)ko, (uint32_t)nf,
                                                       (LDS_AS uint32_t *)s_list[w]);
    if (L.left) {
        if (lane == 0) A.tflag[ti] = 1;
        return;
    }
    if (L.cut && lane == 0) A.bflag[2 * R.buf + 1] = 1;
    if (!kAgain && lane == 0 && is_sampled(r, T.n_req))
        atomicAdd((unsigned long long *)(A.sample + kSampleStride * ti),
                  (unsigned long long)pack_sample(L.np, L.fresh, nf));
    if (lane == 0) {
        RunReq q;
        q.n_full = (uint32_t)nf;
        q.prefix = T.prefix[r];
        q.info = (uint32_t)T.group[r] | ((uint32_t)T.contract[r] << 8) |
                 (A.first[R.first0 + q.prefix] < (uint32_t)r ? 1u << 16 : 0u) |
                 L.np << 24;
        q.dt = T.tick ? (uint32_t)(T.tick[r] - (r > 0 ? T.tick[r - 1] : 0)) : r > 0 ? 1u : 0u;
        q.ko = L.np > 0 ? (uint32_t)ko : 0u;
        q.nn = L.nn;
        q.pad[0] = q.pad[1] = 0u;
        A.req[R.req0 + r] = q;
    }
}

// ------------------------------------------------------------ replay
// The requests of a trace, as one wavefront goes through them: descriptors
// come eight at a time (lane 8 j + k: word k of request 8 b + j), a batch
// ahead, and a request's pieces one request ahead, all by vector loads: a
// scalar load in flight would make every LDS wait wait for it too.
struct Feed {
    const GLOBAL uint32_t *rec;
    const GLOBAL uint2 *piece;
    GLOBAL uint32_t *gbits;      // admitted bits in the workspace (PrefixShield, many prefixes)
    LDS_AS uint32_t *lbits;      // ... or in LDS
    GLOBAL int4 *pr;             // per-request quadruples, or null
    int64_t n;
    int32_t n_words;             // of the admitted bits
    bool in_lds;
};

DEV RunReq unpack(uint32_t rec, uint32_t j) {
    RunReq q;
    const int b = (int)(8u * j);
    q.n_full = DevWave::rdl(rec, b);
    q.info = DevWave::rdl(rec, b + 1);
    q.prefix = DevWave::rdl(rec, b + 2);
    q.dt = DevWave::rdl(rec, b + 3);
    q.nn = DevWave::rdl(rec, b + 5);
    return q;
}
DEV uint32_t load_batch(const Feed &F, int64_t b, uint32_t lane) {
    const int64_t i = 64 * b + lane;
    const uint32_t x = F.rec[i < 8 * F.n ? i : 0];      // (n > 0)
    return i < 8 * F.n ? x : 0u;
}
// (lanes past the last piece read the first one again)
DEV uint2 load_pieces(const Feed &F, uint32_t ko, uint32_t info, uint32_t lane) {
    const GLOBAL uint2 *p = F.piece + (ko + (lane < (info >> 24) ? lane : 0u));
    return make_uint2(p->x, p->y);
}

// All requests; false if the instance is lost to this form.
template <int kPol, bool kLdsBits, class X>
DEV bool all_requests(X &R, const Feed &F) {
    const uint32_t lane = (uint32_t)__lane_id();
    const uint32_t n = (uint32_t)F.n;
    if (n == 0) return true;
    uint32_t cur = load_batch(F, 0, lane), nxt = load_batch(F, 1, lane);
    uint2 pc = load_pieces(F, DevWave::rdl(cur, 4), DevWave::rdl(cur, 1), lane);
    uint32_t word = 0;           // (bits in the workspace: lane 0) admitted bits around q.prefix
    if (kPol == 2 && !kLdsBits && lane == 0) word = F.gbits[DevWave::rdl(cur, 2) >> 5];
    for (uint32_t r = 0; r < n; ++r) {
        const RunReq q = unpack(cur, r & 7u);
        const uint32_t j = (r + 1) & 7u;
        if (__builtin_expect(j == 0, 0)) {
            if (((r + 1) & (X::kFlush - 1u)) == 0) R.flush();
            cur = nxt;
            nxt = load_batch(F, ((int64_t)(r + 1) >> 3) + 1, lane);
        }
        // the next request's pieces (zeros past the last request)
        const uint2 pn = load_pieces(F, DevWave::rdl(cur, (int)(8u * j) + 4), DevWave::rdl(cur, (int)(8u * j) + 1), lane);
        uint32_t np_prefix = 0;
        if (kPol == 2 && !kLdsBits) np_prefix = DevWave::rdl(cur, (int)(8u * j) + 2);
        bool adm = false;
        uint32_t wn = 0;
        if (kPol == 2) {
            if (kLdsBits) word = F.lbits[q.prefix >> 5];
            else if (lane == 0) wn = F.gbits[np_prefix >> 5];
            adm = (DevWave::rfl(word) >> (q.prefix & 31)) & 1u;
        }
        const bool now = R.request(r, q, pc.x, pc.y, adm);
        if (__builtin_expect(R.over != 0, 0)) return false;
        if (kPol == 2) {
            if (now && !adm) {
                word |= 1u << (q.prefix & 31);
                if (kLdsBits) F.lbits[q.prefix >> 5] = word;      // (every lane the same word)
                else if (lane == 0) F.gbits[q.prefix >> 5] = word;
                DevWave::sync();
            }
            if (!kLdsBits) word = (np_prefix >> 5) == (q.prefix >> 5) ? word : wn;
        }
        if (__builtin_expect(F.pr != nullptr, 0)) {      // (every lane the same quadruple)
            GLOBAL int4 *o = F.pr + r;
            o->x = R.last_h;
            o->y = R.last_m;
            o->z = R.last_e;
            o->w = R.last_o;
        }
        pc = pn;
    }
    return true;
}

DEV void clear_bits(const Feed &F) {
    for (int i = (int)__lane_id(); i < F.n_words; i += 64) {
        if (F.in_lds) F.lbits[i] = 0u;
        else F.gbits[i] = 0u;
    }
    DevWave::sync();
    if (!F.in_lds) __threadfence();
}

// stats record: 64 groups x 17 int64, then the instance block
template <class X>
DEV void write_stats(X &R, int64_t n, int G, int64_t *st) {
    const int lane = (int)__lane_id();
    R.flush();
    int64_t *o = st + lane * kGroupFields;
    const bool grp = lane < G;
    const int64_t v[kGroupFields] = {R.c_req, R.c_probe, R.c_hit, R.c_probe - R.c_hit, R.c_probe - R.c_hit - R.c_dup,
                                     R.c_evw, R.c_evc, R.c_promo, R.c_gated, R.c_orph, R.c_dup, R.c_trunc,
                                     n > 0 ? R.raw_debt() : 0, R.d_max, R.d_sum, (int64_t)R.res, (int64_t)R.res_max};
#pragma unroll
    for (int f = 0; f < kGroupFields; ++f) o[f] = grp ? v[f] : 0;
    // evictions of all groups (every group owns its victims)
    int64_t ev = R.c_evw;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1)
        ev += (int64_t)(((uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)((uint64_t)ev >> 32), d) << 32) |
                        (uint32_t)__shfl_xor((int)(uint32_t)(uint64_t)ev, d));
    if (lane == 0) {
        int64_t *qq = st + kInstOffset;
        qq[0] = ev;
        qq[1] = R.c_moves;
        qq[2] = R.c_reins;
        qq[3] = R.c_ghits;
        qq[4] = R.c_gins;
        qq[5] = (int64_t)R.resident;
        qq[6] = (int64_t)R.rmax;
        qq[7] = 0;
    }
}

template <int kPol, bool kK1, bool kLdsBits>
DEV bool replay_one(const RunParams &P, const Feed &F, int64_t *st, LDS_AS uint32_t *lds) {
    DevWave wv;
    RunReplay<DevWave, kPol, kK1> X(P, wv, lds);
    if (kPol == 2) clear_bits(F);
    if (!all_requests<kPol, kLdsBits>(X, F)) return false;
    write_stats(X, F.n, P.G, st);
    return true;
}
// One instance.  False: left to the general kernel.
template <int kPol>
DEV bool replay_policy(const RunParams &P, const Feed &F, int64_t *st, LDS_AS uint32_t *lds) {
    if (kPol == 2 && !F.in_lds)
        return P.K == 1 ? replay_one<kPol, true, false>(P, F, st, lds) : replay_one<kPol, false, false>(P, F, st, lds);
    return P.K == 1 ? replay_one<kPol, true, true>(P, F, st, lds) : replay_one<kPol, false, true>(P, F, st, lds);
}

DEV void replay_instance(const RunsArgs &A, const int32_t *__restrict__ order, uint8_t *ws, int64_t *stats,
                         int32_t *per_req) {
    extern __shared__ __align__(16) uint32_t runs_smem[];
    const int id = order[blockIdx.x];
    if (A.wide && A.done[id]) return;
    const uint32_t pays = !A.wide ? kPaysFirst : *A.n_over <= A.n_cu ? kPaysWideFew : kPaysWideMany;
    if (!(A.pays[id] & pays)) return;
    const DevInst &I = A.inst[id];
    const DevRunTrace &R = A.traces[I.run_trace];
    if (A.tflag[I.run_trace] || A.bflag[2 * R.buf] || A.cmax[I.run_trace] >= I.n_contracts) return;
    const DevTrace &T = A.tr[I.trace];
    LDS_AS uint32_t *lds = (LDS_AS uint32_t *)runs_smem;
    RunParams P;
    P.C = I.capacity;
    P.G = T.n_groups;
    P.K = I.n_contracts;
    P.flags = I.flags;
    P.s_cap = I.s_cap;
    P.g_cap = I.g_cap;
    P.move_thr = I.move_thr;
    P.win = runs_windows(I.policy, I.capacity, A.wide);
    P.eps = I.eps;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        P.rho[c] = I.rho[c];
        P.beta[c] = I.beta[c];
        P.invw[c] = I.invw[c];
    }
    Feed F;
    F.rec = (const GLOBAL uint32_t *)(A.req + R.req0);
    F.piece = (const GLOBAL uint2 *)(A.table + A.bufs[R.buf].tab0);
    F.gbits = (GLOBAL uint32_t *)(ws + I.ws_bits);
    F.in_lds = T.n_prefix <= kRunsLdsPrefix;
    F.n_words = I.n_prefix_words;
    F.lbits = lds + runs_lds_bytes(I.policy, P.win, 0) / 4;
    F.pr = (per_req && I.per_req_off >= 0) ? (GLOBAL int4 *)(per_req + I.per_req_off) : nullptr;
    F.n = T.n_req;
    int64_t *st = (int64_t *)DevWave::hold((uint64_t)(stats + (int64_t)id * kRecordWords));
    int32_t *done = (int32_t *)DevWave::hold((uint64_t)(A.done + id));
    int32_t *over = (int32_t *)DevWave::hold((uint64_t)A.n_over);
    const int32_t route = DevWave::hold(A.wide ? PC_ROUTE_RUNS_WIDE : PC_ROUTE_RUNS);
    bool ok;
    if (I.policy == kLRU) ok = replay_policy<kLRU>(P, F, st, lds);
    else if (I.policy == kS3) ok = replay_policy<kS3>(P, F, st, lds);
    else if (I.policy == kSQ) ok = replay_policy<kSQ>(P, F, st, lds);
    else ok = replay_policy<kPS>(P, F, st, lds);
    if (threadIdx.x == 0) {
        if (ok) *done = route;
        else if (route == PC_ROUTE_RUNS) atomicAdd(over, 1);
    }
}
__global__ __launch_bounds__(64) void runs_replay(RunsArgs A, const int32_t *__restrict__ order, uint8_t *ws,
                                                  int64_t *stats, int32_t *per_req) {
    replay_instance(A, order, ws, stats, per_req);
}
// The same with so many registers asked for that a second wavefront of this
// kernel does not fit on the SIMD (others do): see plan_run_launches.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 1))) void runs_replay_alone(
    RunsArgs A, const int32_t *__restrict__ order, uint8_t *ws, int64_t *stats, int32_t *per_req) {
    replay_instance(A, order, ws, stats, per_req);
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
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&runs_replay),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&runs_replay_alone),
                               hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
}

hipError_t launch_runs_replay(const RunsArgs &A, const int32_t *d_order, int32_t n_launch, int32_t lds_bytes,
                              int32_t alone, uint8_t *ws, int64_t *stats, int32_t *per_req, hipStream_t s) {
    if (alone)
        hipLaunchKernelGGL(runs_replay_alone, dim3((unsigned)n_launch), dim3(64), (size_t)lds_bytes, s, A, d_order,
                           ws, stats, per_req);
    else
        hipLaunchKernelGGL(runs_replay, dim3((unsigned)n_launch), dim3(64), (size_t)lds_bytes, s, A, d_order, ws,
                           stats, per_req);
    return hipGetLastError();
}

}  // namespace pcr
