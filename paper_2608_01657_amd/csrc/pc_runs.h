// pc_runs.h -- replay of one cache instance by one wavefront, on runs of
// blocks instead of single blocks.
//
// The trace analysis (pc_runs.hip) numbers every distinct block key by the
// position of its first occurrence in the key buffer (its id) and cuts every
// request into pieces: maximal stretches of consecutive ids inside which no
// id has a weak link.  The link into id x is weak when some request holds x
// without holding x - 1 right before it; so a request that holds x, and whose
// link is not weak, holds x - 1 as well.  Two facts follow, for any keys at
// all (chained or not):
//   (a) a run [lo, hi) of cached blocks that was taken from one piece meets a
//       request in a leading part [lo, s) only, and inside one piece of it;
//   (b) the blocks of a run that were released together leave the free queue
//       deepest first, so what an eviction takes is a trailing part [s, hi).
// A set of blocks that enters the free queue together therefore stays one
// run of ids for as long as it is cached, and the cache is a short list of
// runs (30-110 for 4,096 blocks of one-touch prompts) with the attributes
// that the policies look at.  Lookup, reclamation and release then cost a
// few wavefront steps for a whole request, with no key compares, no hash
// table and no barriers.
//
// A run is its first id and a word of length (bits 0-15) and attributes:
// owner group (16-21), contract (22-23), retention class (24-25), S3-FIFO
// frequency (26-27), emptied (31); PrefixShield adds the prefix id, S3-FIFO
// the request that pins it, the ghost the sequence of its last id.  Runs
// stand in windows in LDS in free-queue order, 64 to a chunk; a run emptied
// by hits or evictions stays behind (id kNone) until the window is compacted.
//
// What bounds a request is the instruction stream of its one wavefront: about
// 4 cycles an instruction and 20-25 more a branch, with no other wavefront on
// the SIMD to fill them.  So steps look at four chunks at once without a
// branch in between, and what is rare stands behind one common test.
//
// The code is written for one wavefront with uniform control flow: `vu`,
// `vl` and `vb` are a per-lane 32-bit word, 64-bit integer and condition,
// everything else is uniform.  On the device they are the plain types; a
// host build takes 64-lane structures instead and runs the same source on
// the CPU, lane by lane.
//
// An instance that needs more runs than its windows hold is replayed again,
// with windows that take a CU's whole LDS (960 conversation instances 222 ms;
// 281 with the general kernel instead of that); one that needs more than those
// is left to the general kernel (pc_replay.hip).  What the analysis can tell
// is left to it at once: the instances of a trace with a request of more
// pieces than lanes, those with fewer contracts than a request names, and
// those of many short pieces, which the general kernel replays faster
// (runs_pay).
#pragma once
#include <stdint.h>

namespace pcr {

// One request as the trace analysis leaves it: eight words, read by every
// instance of the trace, eight requests to a wavefront load.
struct RunReq {
    uint32_t n_full;     // full blocks
    uint32_t info;       // bits 0-7 group, 8-15 contract, 16: its prefix was referenced before, 24-30 pieces
    uint32_t prefix;
    uint32_t dt;         // ticks since the request before it
    uint32_t ko;         // its pieces start at pieces[ko] of the trace's key buffer
    uint32_t nn;         // blocks that are no duplicates
    uint32_t pad[2];
};
constexpr uint32_t kRunsMaxPieces = 64;      // a lane each; a trace with a request of more is left
// One piece: its first id; its length (bits 0-14, at most 32,767), whether an
// earlier piece of the request holds the same blocks (bit 15: duplicates,
// skipped), and how many blocks that are no duplicates come before it (bits
// 16-31, at most 65,535).  A request fills 32,767 blocks of a cache at most,
// so what the limits cut off is cut off anyway.
struct RunPiece {
    uint32_t id, len;
};
constexpr uint32_t kPieceLen = 0x7FFFu, kPieceDup = 0x8000u;

// Entries of an instance's windows (multiples of 256): of the free queue,
// under S3-FIFO of the small queue, the main queue and the ghost.  At first
// (wide = 0) instances of up to 4,096 blocks fit five to a CU's LDS under any
// policy and larger ones three, since a wavefront on every SIMD is what counts
// for a batch of 1,024; there is room for runs of 3 blocks on average
// (S3-FIFO: 5), above 4,096 blocks for runs of 6 to 11.
struct RunWindows {
    int32_t n[3];
};
constexpr RunWindows runs_windows(int policy, int32_t capacity, int wide) {
    if (wide) {      // one instance to a CU; no window needs more than a run a block, and slack
        const int32_t most = (capacity + 639) / 256 * 256;
        if (policy == 1) return {{most < 4096 ? most : 4096, most < 4864 ? most : 4864, most < 3328 ? most : 3328}};
        const int32_t n = policy == 2 ? 12032 : 18432;
        return {{most < n ? most : n, 0, 0}};
    }
    if (capacity <= 384) return {{512, policy == 1 ? 512 : 0, policy == 1 ? 512 : 0}};
    if (policy == 1) return capacity <= 4096 ? RunWindows{{1024, 768, 768}} : RunWindows{{1280, 2048, 1024}};
    return {{capacity <= 2048 ? 1024 : capacity <= 4096 ? 1536 : 3072, 0, 0}};
}
// Live runs that the first windows are sure to hold (S3-FIFO: by the ghost's).
constexpr int32_t runs_narrow_room(int policy, int32_t capacity) {
    const RunWindows w = runs_windows(policy, capacity, 0);
    return w.n[policy == 1 ? 2 : 0] - 128;
}
// PrefixShield keeps its admitted bits in LDS up to this many prefixes.
constexpr int32_t kRunsLdsPrefix = 1 << 16;
constexpr int32_t kRunsScratch = 192;     // words that single-lane stores spread over
// LDS bytes of one instance: scratch, windows, admitted bits.
constexpr int32_t runs_lds_bytes(int policy, RunWindows w, int64_t n_prefix) {
    const int64_t words = (policy == 1 || policy == 2 ? 3 : 2) * ((int64_t)w.n[0] + w.n[1] + w.n[2]);
    const int64_t bits = policy == 2 && n_prefix <= kRunsLdsPrefix ? (n_prefix + 31) / 32 : 0;
    return (int32_t)(4 * (kRunsScratch + words + bits));
}

// ------------------------------------------------------------ which form
// Sums over a sample of a trace's requests: one of every 64th part of the
// trace, or all (what repeats in a fixed rhythm comes in as often as it is).
struct RunsSample {
    uint32_t n, pieces;       // requests; their pieces
    uint32_t blocks, fresh;   // blocks; pieces that no earlier request holds
};
constexpr int64_t kSamples = 64;
PC_RUNS_FN bool is_sampled(int64_t r, int64_t n_req) {
    const uint32_t part = (uint32_t)((n_req + kSamples - 1) / kSamples), k = (uint32_t)r / part;
    // (2^32 over the golden ratio)
    return (uint32_t)r - k * part == ((k + 1u) * 0x9E3779B1u >> 8) % part;
}
// All four in one word, for one atomic addition a sampled request, each trace's
// word on a line of its own (8 words): additions to one line follow each other,
// some 20 to 40 ns each.  n and fresh take at most 64 and 64 * 64, pieces the
// same, blocks (cut at 65,535 each) less than 2^22.
constexpr int64_t kSampleStride = 8;
PC_RUNS_FN uint64_t pack_sample(uint32_t np, uint32_t fresh, int64_t nf) {
    return 1ull | (uint64_t)np << 7 | (uint64_t)fresh << 20 | (uint64_t)(nf < 65535 ? nf : 65535) << 33;
}
PC_RUNS_FN RunsSample unpack_sample(uint64_t w) {
    return {(uint32_t)w & 0x7Fu, (uint32_t)(w >> 7) & 0x1FFFu, (uint32_t)(w >> 33), (uint32_t)(w >> 20) & 0x1FFFu};
}

// Estimated time of a request (us), by an instance alone on the chip.  On runs
// every piece is compared with every 256 entries of the windows, so many short
// pieces cost more than the blocks that they hold cost the general kernel
// (LRU, C = 4,096, requests of k documents of d blocks, on runs and general
// kernel): k 4, d 16 2.5 and 4.9; k 16, d 16 6.5 and 5.4; k 24, d 4 15 and 5.1;
// k 60, d 1 89 and 5.2 (C = 16,384: 265 and 7.0).  Over 546 such batches of all
// policies the form that these take is at most 1.3 times slower than the
// general kernel (always runs: 38 times).
struct FormTimes {
    float first, wide, general;      // on runs with the first windows, which may turn out too small; the widest
};
//   C      capacity
//   room   blocks that a request may hold
PC_RUNS_FN FormTimes form_times(int policy, int32_t C, int32_t room, int64_t n_req, const RunsSample &q) {
    if (q.n == 0 || q.pieces == 0) return {1.0f, 1.0f, 4.0f};
    const float n = (float)q.n, np = (float)q.pieces / n, nf = (float)q.blocks / n;
    const float cut = nf > (float)room ? (float)room / nf : 1.0f, x = nf * cut / 256.0f;
    // runs in the cache: what fills it, or all that the trace has; on average
    // over a trace that fills it as it goes
    const float total = (float)q.fresh / n * (float)n_req;
    const float fill = (float)C * np / nf, live = fill < total ? fill : total;
    const float mean = live - live * live / (2.0f * (total > 1.0f ? total : 1.0f));
    const float groups = mean > 256.0f ? mean / 256.0f : 1.0f;
    FormTimes t;
    if (policy == 1) {
        t.wide = 1.2f + np * (0.52f * cut + 0.13f * groups);
        t.general = 7.0f + 4.5f * x > 11.5f * x ? 7.0f + 4.5f * x : 11.5f * x;
    } else if (policy == 2) {
        t.wide = 1.5f + np * (0.15f * cut + 0.095f * groups);
        t.general = 6.0f + 8.0f * x > 13.0f * x ? 6.0f + 8.0f * x : 13.0f * x;
    } else {
        t.wide = 1.0f + np * (0.2f * cut + 0.085f * groups);
        t.general = 4.6f + 0.5f * x > 5.1f * x ? 4.6f + 0.5f * x : 5.1f * x;
    }
    t.first = live > (float)runs_narrow_room(policy, C) ? 1.6f * t.wide : t.wide;
    return t;
}
// Which launches on runs an instance is worth: the first; the one with the
// widest windows, a CU to an instance, when all that get there have one at
// once; when they are more (`load`, `rounds`: how many instances of the batch
// share what one alone would have, in the general kernels and with the widest
// windows).
constexpr uint32_t kPaysFirst = 1, kPaysWideFew = 2, kPaysWideMany = 4, kPaysAll = 7;
PC_RUNS_FN uint32_t runs_pay(const FormTimes &t, float load, float rounds) {
    return (t.first <= t.general * load ? kPaysFirst : 0u) | (t.wide <= t.general ? kPaysWideFew : 0u) |
           (t.wide * rounds <= t.general * load ? kPaysWideMany : 0u);
}
// The general kernels begin when the replay on runs has ended, so a batch that
// needs both takes as long as its longest instance on runs (runs_in) and its
// longest in the general kernels (general_in): all in the general kernels
// (general_all), or all on runs that can (runs_all), may be over earlier.
PC_RUNS_FN uint32_t batch_pays(uint32_t pays, float runs_in, float general_in, float runs_all, float general_all) {
    const float both = runs_in + general_in;
    if (general_all < 0.9f * both && general_all <= runs_all) return 0u;
    return runs_all < 0.9f * both ? kPaysAll : pays;
}

// ------------------------------------------------------------ analysis
// What is known of a key buffer when its requests are cut into pieces.
struct RunsBuf {
    const uint32_t *id;       // per position: its id (bit 31 is not part of it)
    const uint32_t *weak;     // bitmap over ids: weak links
    uint32_t *cuts;           // bitmap over ids: links cut for the sake of duplicates
    const uint32_t *start;    // bitmap over positions: request_marks
    uint32_t *piece;          // per position: two words (RunPiece)
};
constexpr uint32_t kRunsResolved = 0x80000000u;    // id[pos] holds the id, not yet the table slot
// Positions whose link is weak for the sake of a request of nf blocks at ko:
// where it starts, and where it ends if it is its trace's last (any other ends
// where the next one starts).  Two traces may cut one key buffer differently
// and keep their pieces in one array; since ends are marked too, requests
// that start at the same position have the same pieces up to where the shorter
// ends.
template <class F>
PC_RUNS_FN void request_marks(int64_t ko, int64_t nf, bool last, int64_t n_keys, F mark) {
    if (nf > 0) mark(ko);
    if (last && ko + nf < n_keys) mark(ko + nf);
}
struct RunsListed {
    uint32_t np, nn;          // pieces; blocks that are no duplicates
    uint32_t fresh;           // pieces that begin with a block first seen in this request
    bool cut;                 // added a cut
    bool left;                // not for this form
};
// The pieces of the request of nf blocks at position ko, by one wavefront;
// `s`: 128 words of LDS.
//
// Where pieces with the same first id differ in length (a document in full
// and its beginning), the longer one is cut where the shorter ends, or it
// could not be told which of its blocks are duplicates.  The first pass finds
// these cuts and the second (kAgain), where there are any, lists every request
// again.  The second adds none and needs none: the first reads `weak`, which
// nobody writes meanwhile, so all of its lists follow from the same links.  A
// block at a new cut has no weak link, so every request that holds it got to
// it through the piece that was cut; so the pieces that begin there are ends
// of pieces with one first id, each cut wherever another of them ends.
template <class W, bool kAgain>
PC_RUNS_FN RunsListed list_request(W &wv, const RunsBuf &B, uint32_t ko, uint32_t nf, typename W::Lds s) {
    using vu = typename W::vu;
    using vb = typename W::vb;
    const vu lane = wv.lane(), zu = wv.vu0(0);
    RunsListed R{0u, nf, 0u, false, false};
    for (uint32_t j0 = 0; j0 < nf; j0 += 64) {
        const vu j = lane + j0;
        const vb in = j < nf;
        const vu x = W::gld(in, B.id, j + ko) & ~kRunsResolved;
        vu links = W::gld(in, B.weak, x >> 5);
        if (kAgain) links = links | W::gld(in, B.cuts, x >> 5);
        const vb cut = in & W::bit(links, x);
        const uint64_t m = W::ballot(cut);
        const vu k = W::mbcnt(m) + R.np;
        const vb keep = cut & (k < 64u);
        W::st(keep, s, k, x);
        W::st(keep, s, k + 64u, j);
        R.np += (uint32_t)W::popc(m);
    }
    W::sync();
    if (R.np > kRunsMaxPieces) {
        R.left = true;
        return R;
    }
    const vb in = lane < R.np;
    const vu pid = W::ld_if(in, s, lane), dep = W::ld_if(in, s, lane + 64u);
    const vu end = W::sel(lane + 1u < R.np, W::next_lane(dep), wv.vu0(nf));
    const vu len = W::sel(in, end - dep, zu);
    vb dup = lane < 0u;
    for (uint32_t i = 0; i + 1 < R.np; ++i) {
        const uint32_t a = W::rdl(pid, (int)i), la = W::rdl(len, (int)i);
        const vb same = in & (lane > i) & (pid == a);
        dup = dup | same;
        const vb differ = same & (len != la);
        if (W::ballot(differ) == 0) continue;
        if (kAgain) {      // cannot happen, see above
            R.left = true;
            return R;
        }
        W::gor_bit(differ, B.cuts, W::vmin(len, wv.vu0(la)) + a);
        R.cut = true;
    }
    // the pieces are kept at the request's own key positions; another trace's
    // request may start (or end) among them when traces overlap.  One that
    // starts at ko itself writes the same pieces there.
    const vu at = lane + ko;
    const vb behind = in & (lane > 0u);
    if (W::ballot(behind & W::bit(W::gld(behind, B.start, at >> 5), at)) != 0) {
        R.left = true;
        return R;
    }
    const vu own = W::sel(dup, zu, len);
    const vu upto = W::scan(own), before = upto - own;
    R.nn = W::rdl(upto, 63);
    R.fresh = (uint32_t)W::popc(W::ballot((own > 0u) & (pid >= ko)));
    W::gst2(in, B.piece, at, pid,
            W::vmin(len, wv.vu0(kPieceLen)) | W::sel(dup, wv.vu0(kPieceDup), zu) |
                (W::vmin(before, wv.vu0(0xFFFFu)) << 16));
    return R;
}

// Replay parameters of one instance (uniform).
struct RunParams {
    int32_t C, G, K, flags;
    int32_t s_cap, g_cap, move_thr;
    RunWindows win;
    int64_t eps;
    int64_t rho[4], beta[4], invw[4];
    int64_t n_req;
};

// `W` supplies the lane types and wavefront operations; kK1: one contract.
template <class W, int kPol, bool kK1>
struct RunReplay {
    using vu = typename W::vu;
    using vl = typename W::vl;
    using vb = typename W::vb;
    using Lds = typename W::Lds;
    static constexpr int LRU = 0, S3 = 1, PS = 2, SQ = 3;
    static constexpr bool kX = kPol == PS || kPol == S3;      // runs carry a third word
    static constexpr bool kQ = kPol == PS || kPol == SQ;      // counts per (group, segment)
    static constexpr uint32_t kLen = 0xFFFFu, kAttr = 0xFFFF0000u;
    static constexpr int kOwnS = 16, kConS = 22, kClsS = 24, kFrqS = 26;
    static constexpr uint32_t kOwnM = 63u << 16, kClsM = 3u << 24;
    static constexpr uint32_t kDead = 0x80000000u;            // word of an emptied run
    static constexpr uint32_t kReuseCls = 2, kNormalCls = 1, kProbCls = 0;
    static constexpr uint32_t kNone = 0xFFFFFFFFu;
    static constexpr int kC = kK1 ? 1 : 4;
    // Entries that a request may need in the queue's window beyond one per
    // piece (hits it releases, parts that the ghost remembers, splits).
    static constexpr uint32_t kSlack = 128;
    static constexpr uint32_t kFlush = 32768;     // requests between flushes of the 32-bit counters
    // Words from one chunk of a window to the next, and to a run's second
    // and third word.
    static constexpr uint32_t kStep = 64 * (kX ? 3 : 2), kW = 64, kXo = 128;

    struct Window {
        Lds p;
        vu cap;                  // entries (uniform; rarely looked at)
        uint32_t tail;           // entries in use
        uint32_t lim;            // compact when the window would grow past this
    };
    // Four chunks (a group) of one word of the runs.
    struct Four {
        vu v[4];
    };

    const RunParams &P;
    W &wv;
    const vu lane;
    const Lds scratch;
    Window q0, q1, gh;           // free queue (S3-FIFO: small, main, ghost)
    uint32_t over;               // not 0: a window was too small, the state is lost

    // the runs that the request meets (lane k: the k-th)
    vu md, mlo, mw, mx, mi;
    uint32_t nm;
    // words of the queue's first group, as the request goes (not S3-FIFO)
    Four lo4, w4;

    // uniform state (what only vector instructions use stands in vector
    // registers: scalar ones are what a request runs out of)
    int32_t resident;
    int32_t s_size, s_unp, m_unp;
    uint32_t gseq;
    vu rmax, n_moves, n_reins, n_ghits, n_gins;          // since the last flush (rmax aside)
    vl c_moves, c_reins, c_ghits, c_gins;
    vl rho[kC], beta[kC];
    int32_t last_h, last_m, last_e, last_o;
    // lane x = group x
    vl E[kC];                    // effective balances at tprev (Eq. 1)
    vl d_max, d_sum;
    vu cnt0, cnt1, cnt2;         // queued blocks per segment (kQ)
    vu res, res_max;
    vu evw, n_req, n_probe, n_hit, n_evc;         // since the last flush
    vl c_evw, c_req, c_probe, c_hit, c_evc, c_dup, c_trunc, c_promo, c_gated, c_orph;

    static PC_RUNS_FN uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
    static PC_RUNS_FN uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
    PC_RUNS_FN int K() const { return kK1 ? 1 : P.K; }

    PC_RUNS_FN RunReplay(const RunParams &p, W &w, Lds base)
        : P(p), wv(w), lane(w.lane()), scratch(base) {
        Lds at = base + (uint32_t)kRunsScratch;
        at = open(q0, at, (uint32_t)P.win.n[0]);
        if (kPol == S3) {
            at = open(q1, at, (uint32_t)P.win.n[1]);
            open(gh, at, (uint32_t)P.win.n[2]);
        }
        over = 0;
        resident = 0;
        s_size = s_unp = m_unp = 0;
        gseq = 0;
        last_h = last_m = last_e = last_o = 0;
        nm = 0;
        const vl z = wv.vl0(0);
        const vu zu = wv.vu0(0);
        md = mlo = mw = mx = mi = zu;
#pragma unroll
        for (int c = 0; c < 4; ++c) lo4.v[c] = w4.v[c] = zu;
#pragma unroll
        for (int c = 0; c < kC; ++c) {
            E[c] = wv.vl0(c < P.K ? P.beta[c] : 0);
            rho[c] = W::hold(wv.vl0(P.rho[c]));
            beta[c] = W::hold(wv.vl0(P.beta[c]));
        }
        rmax = n_moves = n_reins = n_ghits = n_gins = W::hold(zu);
        c_moves = c_reins = c_ghits = c_gins = z;
        d_max = d_sum = z;
        cnt0 = cnt1 = cnt2 = res = res_max = zu;
        evw = n_req = n_probe = n_hit = n_evc = zu;
        c_evw = c_req = c_probe = c_hit = c_evc = c_dup = c_trunc = c_promo = c_gated = c_orph = z;
    }
    // Entries past the tail are emptied runs.
    PC_RUNS_FN Lds open(Window &r, Lds at, uint32_t n) {
        r.p = at;
        r.cap = W::hold(wv.vu0(n));
        r.tail = 0;
        r.lim = 64;
        for (uint32_t b = 0; b < n; b += 64) {
            W::st_all(r.p, lane + entry(b), wv.vu0(kNone));
            W::st_all(r.p, lane + (entry(b) + kW), wv.vu0(kDead));
        }
        W::sync();
        return at + (kX ? 3u : 2u) * n;
    }
    // first word of the entry at a window position
    static PC_RUNS_FN uint32_t entry(uint32_t pos) { return pos + (pos >> 6) * (kStep - 64u); }

    // ------------------------------------------------------------ debts
    // Eqs. 1 and 3: balances move on by dt ticks.  The lazy refill of Eq. 1
    // composes exactly: min(beta, min(beta, B + rho d1) + rho d2) =
    // min(beta, B + rho (d1 + d2)), so the balances are kept at the last
    // tick and every request adds one uniform amount.  2^62 stands for any
    // amount that certainly reaches beta (balances stay above -2^61).
    PC_RUNS_FN void refill(uint32_t dt) {
#pragma unroll
        for (int c = 0; c < kC; ++c)
            if (c < K()) {
                vl inc = rho[c];
                // (rho <= 2^40 and dt < 2^32: only a product past 2^64 wraps)
                if (W::unlikely(dt != 1)) inc = W::mul_sat62(inc, dt);
                E[c] = W::vmin(E[c] + inc, beta[c]);
            }
    }
    PC_RUNS_FN vl raw_debt() const {
        vl d = W::vmax(-E[0], (int64_t)0);
#pragma unroll
        for (int c = 1; c < kC; ++c)
            if (c < P.K) d = d + W::vmax(-E[c], (int64_t)0);
        return d;
    }
    // Eq. 5 (1/w_c in Q16) and Eq. 8's decrement
    PC_RUNS_FN void norm_debt(vl &d, vl &dec) const {
        if (kK1) {     // w = 1: a block is a block
            d = W::vmax(-E[0], (int64_t)0);
            dec = wv.vl0(65536);
            return;
        }
        d = wv.vl0(0);
        dec = wv.vl0(0);
#pragma unroll
        for (int c = 0; c < kC; ++c)
            if (c < P.K) {
                const vb neg = E[c] < (int64_t)0;
                d = d + W::sel(neg, W::mul_shr16(-E[c], P.invw[c]), wv.vl0(0));
                const vb take = neg & ((dec == (int64_t)0) | (wv.vl0(P.invw[c]) < dec));
                dec = W::sel(take, wv.vl0(P.invw[c]), dec);
            }
    }

    // ------------------------------------------------------------ windows
    PC_RUNS_FN static uint32_t u_owner(uint32_t w) { return (w >> kOwnS) & 63u; }
    PC_RUNS_FN static uint32_t u_cls(uint32_t w) { return (w >> kClsS) & 3u; }

    // word `off` of the four chunks from position b (a multiple of 256) on
    PC_RUNS_FN Four load4(const Window &r, uint32_t b, uint32_t off) const {
        Four f;
        W::sync();
        const vu at = lane + (entry(b) + off);
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) f.v[c] = W::ld(r.p + c * kStep, at);
        return f;
    }
    PC_RUNS_FN void store(Window &r, uint32_t b, uint32_t c, uint32_t off, vu x) {
        W::st_all(r.p + c * kStep, lane + (entry(b) + off), x);
    }
    // Words of one entry, by lane 0 (the others write words of their own in
    // scratch, so that no execution mask changes).
    PC_RUNS_FN void put2(const Window &r, uint32_t at, uint32_t lo, uint32_t w) {
        wv.template st1<2>(r.p, at, scratch, lo, w, 0u);
    }
    PC_RUNS_FN void put3(const Window &r, uint32_t at, uint32_t lo, uint32_t w, uint32_t x) {
        wv.template st1<kX ? 3 : 2>(r.p, at, scratch, lo, w, x);
    }
    PC_RUNS_FN void put_at(Lds p, uint32_t at, uint32_t lo, uint32_t w, uint32_t x) {
        wv.template st1<3>(p, at, scratch, lo, w, x);
    }
    PC_RUNS_FN void push(Window &r, uint32_t lo, uint32_t w, uint32_t x) {
        put3(r, entry(r.tail), lo, w, x);
        r.tail += 1;
    }

    // Live runs move to the front of the window, in order; the rest of it is
    // emptied.
    PC_RUNS_FN void compact(Window &r) {
        uint32_t nw = 0;
        const uint32_t nc = (r.tail + 63u) >> 6;
        for (uint32_t c = 0; c < nc; ++c) {
            W::sync();
            const vu at = lane + c * kStep;
            const vu lo = W::ld(r.p, at), w = W::ld(r.p + kW, at);
            vu x = w;
            if (kX) x = W::ld(r.p + kXo, at);
            const vb live = lo != kNone;
            const uint64_t m = W::ballot(live);
            const vu pos = W::mbcnt(m) + nw;
            const vu to = pos + (pos >> 6) * (kStep - 64u);
            W::st(live, r.p, to, lo);
            W::st(live, r.p + kW, to, w);
            if (kX) W::st(live, r.p + kXo, to, x);
            nw += (uint32_t)W::popc(m);
        }
        W::sync();
        for (uint32_t c = nw >> 6; c < nc; ++c) {
            const vb past = lane + 64u * c >= nw;
            const vu at = lane + c * kStep;
            W::st(past, r.p, at, wv.vu0(kNone));
            W::st(past, r.p + kW, at, wv.vu0(kDead));
        }
        W::sync();
        r.tail = nw;
        // a scan pays per 256 entries and a compaction per 64: room for 32
        // entries at least, and not past a group that the live runs leave
        r.lim = umin(umax((nw + 32u + 63u) & ~63u, umin((nw + 255u) & ~255u, nw + 128u)), W::uni(r.cap) - kSlack);
    }
    // Room for k more entries, and kSlack behind them, compacting if need be.
    PC_RUNS_FN bool room_for(Window &r, uint32_t k) {
        if (W::likely(r.tail + k <= r.lim)) return true;
        compact(r);
        const uint32_t most = W::uni(r.cap) - kSlack;
        if (r.tail + k > most) return false;
        r.lim = umax(r.lim, umin(r.tail + k + 32u, most));
        return true;
    }
    // The entry at `pos` is needed twice: everything behind it moves up by one.
    PC_RUNS_FN void open_gap(Window &r, uint32_t pos) {
        uint32_t e = r.tail;                 // entries [pos, e) still to move
        while (e > pos) {
            const uint32_t b = e - pos > 64u ? e - 64u : pos;
            W::sync();
            const vu from = lane + b, to = from + 1u;
            const vb in = from < e;
            const vu fa = from + (from >> 6) * (kStep - 64u), ta = to + (to >> 6) * (kStep - 64u);
            const vu lo = W::ld_if(in, r.p, fa), w = W::ld_if(in, r.p + kW, fa), x = W::ld_if(in, r.p + kXo, fa);
            W::st(in, r.p, ta, lo);
            W::st(in, r.p + kW, ta, w);
            W::st(in, r.p + kXo, ta, x);
            e = b;
        }
        W::sync();
        r.tail += 1;
    }

    // d more (or, as a two's complement, fewer) blocks in a queue
    PC_RUNS_FN void count_queue(vu is_owner, uint32_t seg, uint32_t d) {
        cnt0 = W::mad01(is_owner, kPol == SQ || seg == 0 ? d : 0u, cnt0);
        if (kPol == PS) {
            cnt1 = W::mad01(is_owner, seg == 1 ? d : 0u, cnt1);
            cnt2 = W::mad01(is_owner, seg == 2 ? d : 0u, cnt2);
        }
    }
    PC_RUNS_FN vu is_lane(uint32_t l) const { return W::sel(lane == l, wv.vu0(1), wv.vu0(0)); }
    PC_RUNS_FN uint32_t seg_of(uint32_t w) const {
        return (kPol == PS && !(P.flags & 1)) ? u_cls(w) : 0u;
    }
    PC_RUNS_FN void victims(vu is_owner, uint32_t n) {
        const vu t = W::mad01(is_owner, n, wv.vu0(0));
        evw = evw + t;
        res = res - t;
    }

    // k victims from the queue, oldest first: those whose word, under `mask`,
    // is `pat` (owner x >= 0, or any owner).
    PC_RUNS_FN void take(uint32_t mask, uint32_t pat, int32_t x, uint32_t seg, uint32_t k) {
        uint32_t rem = k;
        uint32_t b = 0;
        for (;;) {
            take_chunk<0>(b, mask, pat, x, rem);
            if (W::likely(rem == 0)) break;
            b += 256;
            if (W::unlikely(b >= q0.tail)) { over = 1; rem = 0; break; }   // cannot happen: the counts say that the queue holds k
            lo4 = load4(q0, b, 0);
            w4 = load4(q0, b, kW);
        }
        if (W::unlikely(b)) reload();
        if (kQ && x >= 0) {
            const vu o = is_lane((uint32_t)x);
            victims(o, k);
            count_queue(o, seg, 0u - k);
        }
        resident -= (int32_t)k;
    }
    // ... from chunk c of the group at b on.  A prefix sum over the chunk tells
    // how much of every run goes: cheaper than two runs one by one.
    template <int c>
    PC_RUNS_FN void take_chunk(uint32_t b, uint32_t mask, uint32_t pat, int32_t x, uint32_t &rem) {
        const vb in = (w4.v[c] & (mask | kDead)) == pat;
        if (W::ballot(in) != 0) {
            const vu len = W::sel(in, w4.v[c] & kLen, wv.vu0(0));
            const vu upto = W::scan(len), before = upto - len;
            const vu tk = W::sel(before < rem, W::vmin(len, wv.vu0(rem) - before), wv.vu0(0));
            const vb all = in & (tk == len);
            const uint32_t tot = W::rdl(upto, 63);
            if (!(kQ && x >= 0))
                for (uint64_t vm = W::ballot(tk > 0u); vm; vm &= vm - 1) {
                    const int l = W::ffs(vm);
                    const uint32_t wl = W::rdl(w4.v[c], l), n = W::rdl(tk, l);
                    const vu o = is_lane(u_owner(wl));
                    victims(o, n);
                    if (kQ) count_queue(o, seg_of(wl), 0u - n);
                }
            lo4.v[c] = W::sel(all, wv.vu0(kNone), lo4.v[c]);
            w4.v[c] = W::sel(all, wv.vu0(kDead), w4.v[c] - tk);
            store(q0, b, c, 0, lo4.v[c]);
            store(q0, b, c, kW, w4.v[c]);
            rem = rem > tot ? rem - tot : 0u;
            if (W::likely(rem == 0)) return;
        }
        if constexpr (c < 3) take_chunk<c + 1>(b, mask, pat, x, rem);
    }
    // the queue's first group again
    PC_RUNS_FN void reload() {
        W::sync();
        lo4 = load4(q0, 0, 0);
        w4 = load4(q0, 0, kW);
    }
    // Window position of the oldest live run that matches.
    PC_RUNS_FN uint32_t head_pos(uint32_t mask, uint32_t pat) {
        W::sync();
        const uint32_t nc = (q0.tail + 63u) >> 6;
        for (uint32_t c = 0; c < nc; ++c) {
            const vu w = W::ld(q0.p + kW, lane + c * kStep);
            const uint64_t m = W::ballot((w & (mask | kDead)) == pat);
            if (m) return 64u * c + (uint32_t)W::ffs(m);
        }
        return kNone;
    }
    // Alg. 2 (Eqs. 5-9): runs of victims from the group with the largest
    // projected debt, one (group, segment) queue at a time.  A take that ends
    // with its queue leaves the group in the lead with the rest of its run of
    // wins, so the next turn goes on with the group's next segment.
    PC_RUNS_FN void evict_ps(uint32_t e) {
        const bool seg3 = !(P.flags & 1);
        vl Pd, D;
        norm_debt(Pd, D);
        uint32_t rem = e;
        for (;;) {
            const vb own = (cnt0 | cnt1 | cnt2) > 0u;
            const uint64_t Em = W::ballot(own & (Pd > P.eps));         // Eq. 6
            if (W::unlikely(Em == 0)) break;
            // Eq. 7 among the first and the last of them, or all
            int gs = W::ffs(Em);
            const int l2 = 63 - W::clz(Em);
            int64_t pg = W::rdl64(Pd, gs), p2 = W::rdl64(Pd, l2);
            if (p2 > pg) {
                const int64_t t = pg;
                pg = p2;
                p2 = t;
                gs = l2;
            }
            if (W::popc(Em) != 2) {
                if (W::likely(W::popc(Em) == 1)) {
                    p2 = -1;
                } else {
                    const vl in = W::sel(W::of_mask(Em), Pd, wv.vl0(-1));
                    pg = W::wmax64(in);
                    gs = W::ffs(W::ballot(in == pg));
                    p2 = W::wmax64(W::sel(lane != (uint32_t)gs, in, wv.vl0(-1)));
                }
            }
            if (W::unlikely(p2 == pg)) gs = tie_break(W::ballot(Pd == pg) & Em, seg3);
            const int64_t thr = p2 > P.eps ? p2 : P.eps;
            const int64_t dg = kK1 ? 65536 : W::rdl64(D, gs);
            if (!kK1 && dg <= 0) { over = 1; return; }    // cannot happen: an indebted group has a decrement
            // the group keeps winning strictly while P - i D > max(second, eps)
            const uint32_t c0 = W::rdl(cnt0, gs), c1 = W::rdl(cnt1, gs), c2 = W::rdl(cnt2, gs);
            const uint32_t seg = c0 ? 0u : c1 ? 1u : 2u, cs = c0 ? c0 : c1 ? c1 : c2;
            uint32_t k = umin(cs, rem);
            const uint64_t num = (uint64_t)(pg - thr) + (uint64_t)dg - 1;    // pg >= thr
            const uint64_t wins = kK1 ? num >> 16 : W::udiv(num, (uint64_t)dg);
            if (wins < k) k = wins ? (uint32_t)wins : 1u;
            const uint32_t mask = seg3 ? kOwnM | kClsM : kOwnM;
            take(mask, ((uint32_t)gs << kOwnS) | (seg << kClsS), gs, seg, k);
            rem -= k;
            if (W::likely(rem == 0) || over) return;
            const vl np = Pd - (int64_t)k * dg;
            Pd = W::sel(lane == (uint32_t)gs, W::vmax(np, (int64_t)0), Pd);
        }
        // no indebted candidate owner: global segment order (Eq. 9 fallback)
        for (uint32_t s = 0; s < 3 && rem > 0 && !over; ++s) {
            const uint32_t tot = W::wsum(s == 0 ? cnt0 : s == 1 ? cnt1 : cnt2);
            const uint32_t tk = umin(tot, rem);
            if (tk > 0) take(seg3 ? kClsM : 0u, s << kClsS, -1, s, tk);
            rem -= tk;
        }
        if (rem > 0) over = 1;
    }
    // Ties in projected debt: lowest non-empty segment, then the oldest head.
    PC_RUNS_FN int tie_break(uint64_t tied, bool seg3) {
        uint32_t seg = 0;
        if (seg3) {
            const uint64_t s0 = W::ballot(cnt0 > 0u) & tied, s1 = W::ballot(cnt1 > 0u) & tied;
            if (s0) tied = s0;
            else if (s1) { tied = s1; seg = 1; }
            else seg = 2;
        }
        int gs = W::ffs(tied);
        if (tied & (tied - 1)) {
            uint32_t best = kNone;
            for (uint64_t tm = tied; tm; tm &= tm - 1) {
                const int x = W::ffs(tm);
                const uint32_t hp = head_pos(seg3 ? kOwnM | kClsM : kOwnM, ((uint32_t)x << kOwnS) | (seg << kClsS));
                if (hp < best) { best = hp; gs = x; }
            }
        }
        return gs;
    }

    // ------------------------------------------------------------ S3-FIFO
    // A queue's runs that the request does not pin, oldest first, one chunk
    // at a time in registers; at the end of a chunk it is read again, for
    // what was appended to it meanwhile, before the next one.
    struct Cursor {
        vu lo, w, x;
        uint64_t m;
        uint32_t c;
    };
    PC_RUNS_FN void load(const Window &r, Cursor &q) const {
        W::sync();
        const vu at = lane + q.c * kStep;
        q.lo = W::ld(r.p, at);
        q.w = W::ld(r.p + kW, at);
        q.x = W::ld(r.p + kXo, at);
    }
    PC_RUNS_FN void choose(uint32_t pin, Cursor &q) const {
        q.m = W::ballot(q.x != pin) & W::ballot(q.lo != kNone);
    }
    // The next chunk with such a run; there is one (the counts of blocks that
    // are not pinned say so).
    template <bool kSmall>
    PC_RUNS_FN void advance(const Window &r, uint32_t pin, Cursor &q, uint32_t &rem) {
        if (kSmall) write_back(q);
        load(r, q);
        choose(pin, q);
        while (q.m == 0) {
            q.c += 1;
            if (64u * q.c >= r.tail) {      // cannot happen
                over = 1;
                rem = 0;
                q.c = 0;
                q.m = 1;
                return;
            }
            load(r, q);
            choose(pin, q);
        }
    }
    // The deepest k blocks of the run in lane l (word w, first id lo) leave it.
    // The small queue's chunk, which nothing is appended to meanwhile, is
    // changed in registers and written back at its end; the main queue's in
    // the window.
    PC_RUNS_FN void write_back(const Cursor &q) const {
        const vu at = lane + q.c * kStep;
        W::st_all(q0.p, at, q.lo);
        W::st_all(q0.p + kW, at, q.w);
        W::sync();
    }
    template <bool kSmall>
    PC_RUNS_FN void shorten(Cursor &q, int l, uint32_t lo, uint32_t w, uint32_t k) {
        const bool all = k == (w & kLen);
        const uint32_t nw = all ? kDead : w - k;
        q.w = W::setlane(q.w, l, nw);
        if (kSmall) q.lo = W::setlane(q.lo, l, all ? kNone : lo);
        else put2(q1, entry(64u * q.c) + (uint32_t)l, all ? kNone : lo, nw);
        q.m = all ? q.m & (q.m - 1) : q.m;
    }
    // S, M: the first chunks of the small and the main queue, as they are.
    // Whether a run moves on or leaves is told by selects: a step has one
    // branch, for the queue that it looks at.
    PC_RUNS_FN void evict_s3(uint32_t e, uint32_t pin, Cursor &S, Cursor &M) {
        uint32_t rem = e;
        const uint32_t tail = q1.tail;
        if (W::unlikely(!room_for(q1, 32) || !ghost_room(32))) { over = 1; return; }
        if (W::unlikely(q1.tail != tail)) load(q1, M);       // (compacted)
        choose(pin, S);
        choose(pin, M);
        uint32_t steps = 32 + kSlack / 2;       // each appends a run to either window at most
        const uint32_t ghost = P.g_cap > 0 ? 1u : 0u;
        do {
            if (W::unlikely(--steps == 0)) {
                if (!room_for(q1, 1) || !ghost_room(1)) { over = 1; rem = 0; }
                M.c = 0;         // (positions changed)
                M.m = 0;
                steps = kSlack / 2;
            }
            // blocks of the small queue (deepest first) that go before the
            // one-at-a-time rule would look at the main queue
            const int32_t la = s_size - P.s_cap + 1 < s_unp ? s_size - P.s_cap + 1 : s_unp;
            const int32_t none = m_unp == 0 ? 1 : 0;
            if (W::likely((la > none ? la : none) > 0)) {
                if (W::unlikely(S.m == 0)) advance<true>(q0, pin, S, rem);
                const int l = W::ffs(S.m);
                const uint32_t lo = W::rdl(S.lo, l), w = W::rdl(S.w, l), len = w & kLen;
                // (the first move gives the main queue an unpinned block)
                const bool mv = (int32_t)((w >> kFrqS) & 3u) >= P.move_thr;
                const uint32_t few = (uint32_t)(mv ? (m_unp == 0 && la < 1 ? 1 : la) : (m_unp > 0 ? la : 0x7FFFFFFF));
                // (kept apart: three minima in a row become one vector
                // instruction, and what depends on it moves to vector registers)
                uint32_t k = W::keep(umin(len, few));
                k = mv ? k : umin(k, rem);
                const uint32_t gone = mv ? 0u : k;
                const Lds to = mv ? q1.p : gh.p;
                put_at(to, entry(mv ? q1.tail : gh.tail), lo + len - k,
                       mv ? k | (w & kAttr & ~(3u << kFrqS)) : k, mv ? pin - 1u : gseq);
                q1.tail += mv ? 1u : 0u;
                gh.tail += mv ? 0u : ghost;      // (without a ghost nothing reads what is there)
                m_unp += (int32_t)(k - gone);
                gseq += gone;
                n_moves = n_moves + (k - gone);
                n_gins = n_gins + gone;
                s_size -= (int32_t)k;
                s_unp -= (int32_t)k;
                shorten<true>(S, l, lo, w, k);
                victims(is_lane(u_owner(w)), gone);
                rem -= gone;
            } else {
                if (W::unlikely(M.m == 0)) advance<false>(q1, pin, M, rem);
                const int l = W::ffs(M.m);
                const uint32_t lo = W::rdl(M.lo, l), w = W::rdl(M.w, l), len = w & kLen;
                const bool mv = ((w >> kFrqS) & 3u) != 0;
                const uint32_t k = mv ? len : umin(W::keep(umin(len, rem)), (uint32_t)m_unp);
                const uint32_t gone = mv ? 0u : k;
                shorten<false>(M, l, lo, w, k);
                // (what leaves from here is written nowhere)
                put_at(mv ? q1.p : scratch, mv ? entry(q1.tail) : 0u, lo, w - (1u << kFrqS), pin - 1u);
                q1.tail += mv ? 1u : 0u;
                n_reins = n_reins + (k - gone);
                m_unp -= (int32_t)gone;
                victims(is_lane(u_owner(w)), gone);
                rem -= gone;
            }
        } while (rem > 0);
        write_back(S);
        resident -= (int32_t)e;
    }
    // Room for k more ghost runs: ids that have left the ghost (older than
    // the last g_cap insertions; a run's deepest ids went in first) go first.
    PC_RUNS_FN bool ghost_room(uint32_t k) {
        if (W::likely(gh.tail + k <= gh.lim)) return true;
        W::sync();
        const uint32_t nc = (gh.tail + 63u) >> 6;
        for (uint32_t c = 0; c < nc; ++c) {
            const vu at = lane + c * kStep;
            const vu lo = W::ld(gh.p, at), w = W::ld(gh.p + kW, at), base = W::ld(gh.p + kXo, at);
            const vu age = wv.vu0(gseq - (uint32_t)P.g_cap) - base;     // signed
            const vu ex = W::sel((age >> 31) > 0u, wv.vu0(0), W::vmin(age, w & kLen));
            const vb gone = ex == (w & kLen);
            W::st_all(gh.p, at, W::sel(gone, wv.vu0(kNone), lo));
            W::st_all(gh.p + kW, at, W::sel(gone, wv.vu0(kDead), w - ex));
            W::st_all(gh.p + kXo, at, base + ex);
        }
        return room_for(gh, k);
    }

    // ------------------------------------------------------------ lookup
    PC_RUNS_FN void file(uint32_t d, uint32_t lo, uint32_t w, uint32_t x, uint32_t i) {
        if (W::unlikely(nm >= 64u)) { over = 1; return; }
        md = W::setlane(md, (int)nm, d);
        mlo = W::setlane(mlo, (int)nm, lo);
        mw = W::setlane(mw, (int)nm, w);
        if (kX) mx = W::setlane(mx, (int)nm, x);
        mi = W::setlane(mi, (int)nm, i);
        nm += 1;
    }
    // Pieces [pa, pa + pl) that meet a run of the group, as a mask.
    PC_RUNS_FN uint64_t meets(const Four &lo, uint32_t np, vu pa, vu pl) const {
        uint64_t pm = 0;
        uint32_t i = 0;
        do {
            const uint32_t a = W::rdl(pa, (int)i), L = W::rdl(pl, (int)i);
            const uint64_t any = (W::ballot(lo.v[0] - a < L) | W::ballot(lo.v[1] - a < L)) |
                                 (W::ballot(lo.v[2] - a < L) | W::ballot(lo.v[3] - a < L));
            pm |= any ? 1ull << i : 0ull;
        } while (++i < np);
        return pm;
    }
    // The same for S3-FIFO's three windows at once (`far`: of the ghost only
    // whether; what an eviction of this request adds there meets no piece of it).
    PC_RUNS_FN void meets3(const Four &a4, const Four &b4, const Four &c4, uint32_t np, vu pa, vu pl, uint64_t &pa4,
                           uint64_t &pb4, bool &far) const {
        uint64_t ma = 0, mb = 0, mc = 0;
        uint32_t i = 0;
        do {
            const uint32_t a = W::rdl(pa, (int)i), L = W::rdl(pl, (int)i);
            const uint64_t x = (W::ballot(a4.v[0] - a < L) | W::ballot(a4.v[1] - a < L)) |
                               (W::ballot(a4.v[2] - a < L) | W::ballot(a4.v[3] - a < L));
            const uint64_t y = (W::ballot(b4.v[0] - a < L) | W::ballot(b4.v[1] - a < L)) |
                               (W::ballot(b4.v[2] - a < L) | W::ballot(b4.v[3] - a < L));
            mc |= (W::ballot(c4.v[0] - a < L) | W::ballot(c4.v[1] - a < L)) |
                  (W::ballot(c4.v[2] - a < L) | W::ballot(c4.v[3] - a < L));
            ma |= x ? 1ull << i : 0ull;
            mb |= y ? 1ull << i : 0ull;
        } while (++i < np);
        pa4 = ma;
        pb4 = mb;
        far = mc != 0;
    }
    // Runs of window r, group b (ids lo), that the pieces of mask pm meet:
    // their leading part is filed with its depth in the request and taken off
    // the run (kKeep: left there, its position and window filed).  By (a) at
    // the top a run meets one piece at most.
    template <bool kKeep, bool kGhost>
    PC_RUNS_FN void meet(Window &r, uint32_t b, Four &lo, uint64_t pm, uint32_t ringbit, vu pa, vu pl, vu pc,
                         uint32_t &found, uint32_t &far) {
        for (; pm; pm &= pm - 1) {
            const int i = W::ffs(pm);
            const uint32_t a = W::rdl(pa, i), L = W::rdl(pl, i), depth = W::rdl(pc, i);
#pragma unroll
            for (uint32_t c = 0; c < 4; ++c) {
                uint64_t m = W::ballot(lo.v[c] - a < L);
                if (m == 0) continue;
                const vu at = lane + (entry(b) + c * kStep);
                vu w = W::ld(r.p + kW, at), x = w;
                if (kX && !kKeep) x = W::ld(r.p + kXo, at);
                do {
                    const int l = W::ffs(m);
                    m &= m - 1;
                    const uint32_t el = W::rdl(lo.v[c], l), ew = W::rdl(w, l);
                    uint32_t len = ew & kLen;
                    if (kGhost) {       // (its last ids may have left the ghost)
                        const int32_t age = (int32_t)(gseq - (uint32_t)P.g_cap - W::rdl(x, l));
                        if (age > 0) len -= umin((uint32_t)age, len);
                        if (len == 0) continue;
                    }
                    const uint32_t ov = umin(len, a + L - el), d = depth + (el - a);
                    const uint32_t pos = b + 64u * c + (uint32_t)l;
                    file(d, el, (ew & kAttr) | ov, kKeep ? pos << 1 | ringbit : kX ? W::rdl(x, l) : 0u, (uint32_t)i);
                    found += ov;
                    far = umax(far, d + ov);
                    if (!kKeep) {
                        const bool rest = (ew & kLen) != ov;
                        lo.v[c] = W::setlane(lo.v[c], l, rest ? el + ov : kNone);
                        w = W::setlane(w, l, rest ? ew - ov : kDead);
                        if (kQ) count_queue(is_lane(u_owner(ew)), seg_of(ew), 0u - ov);
                    }
                } while (m);
                if (!kKeep) {
                    store(r, b, c, 0, lo.v[c]);
                    store(r, b, c, kW, w);
                    if (!kGhost && b == 0) w4.v[c] = w;
                }
            }
        }
    }
    // All groups of a window from position b on.
    template <bool kKeep, bool kGhost>
    PC_RUNS_FN void meet_from(Window &r, uint32_t b, uint32_t ringbit, uint32_t np, vu pa, vu pl, vu pc,
                              uint32_t &found, uint32_t &far) {
        for (; b < r.tail; b += 256) {
            Four lo = load4(r, b, 0);
            const uint64_t pm = meets(lo, np, pa, pl);
            if (W::unlikely(pm != 0)) meet<kKeep, kGhost>(r, b, lo, pm, ringbit, pa, pl, pc, found, far);
        }
    }

    // ------------------------------------------------------------ request
    // `pid`, `plen`: the request's pieces as stored, lane i piece i (i < np).
    // `adm`: its prefix was admitted before; returns whether it is now.
    // With `over` set, the instance is lost to this form.
    PC_RUNS_FN bool request(uint32_t r, const RunReq &q, vu pid, vu plen, bool adm) {
        const uint32_t g = q.info & 0xFFu, c = (q.info >> 8) & 0xFFu;
        const uint32_t np = q.info >> 24;
        // (the only place that compacts the free queue; S3-FIFO's main queue
        // and ghost are looked at where they grow)
        if (W::unlikely(q0.tail + np > q0.lim) && !room_for(q0, np)) { over = 1; return adm; }
        // S3-FIFO: ids of the first groups of the main queue and the ghost, and
        // the first chunks of the two queues, for the eviction (loaded here,
        // so that it need not wait for them)
        Four m4, g4;
        Cursor S, M;
        if (kPol != S3) {
            reload();
        } else {
            lo4 = load4(q0, 0, 0);
            m4 = load4(q1, 0, 0);
            g4 = load4(gh, 0, 0);
            S.c = M.c = 0;
            load(q0, S);
            load(q1, M);
        }
        const uint32_t gtail = kPol == S3 ? gh.tail : 0u;
        refill(q.dt);
        const uint32_t room = (uint32_t)(kPol == SQ ? P.C / P.G : P.C);
        const uint32_t n = umin(q.n_full, room);
        const vu me = is_lane(g);
        const vu zu = wv.vu0(0);

        // pieces, their lengths without the duplicates, cut to n blocks
        const vb real = lane < np;
        vu pl = W::sel(real & ((plen & kPieceDup) == 0u), plen & kPieceLen, zu);
        const vu pc = plen >> 16;
        uint32_t nn = q.nn;          // blocks that are no duplicates
        if (W::unlikely(n != q.n_full)) {
            const vu raw = W::sel(real, plen & kPieceLen, zu);
            const vu start = W::scan(raw) - raw;
            pl = W::sel(start < n, W::vmin(pl, wv.vu0(n) - start), zu);
            nn = W::wsum(pl);
        }

        // ---- lookup
        nm = 0;
        uint32_t found = 0, far = 0;
        bool ghosts = false;         // S3-FIFO: the ghost may remember blocks of the request
        {
            if (kPol == S3) {
                uint64_t pm, pm1;
                meets3(lo4, m4, g4, np, pid, pl, pm, pm1, ghosts);
                if (W::unlikely((pm | pm1) != 0)) {
                    meet<true, false>(q0, 0, lo4, pm, 0, pid, pl, pc, found, far);
                    meet<true, false>(q1, 0, m4, pm1, 1, pid, pl, pc, found, far);
                }
                if (W::unlikely(umax(q0.tail, q1.tail) > 256)) {
                    meet_from<true, false>(q0, 256, 0, np, pid, pl, pc, found, far);
                    meet_from<true, false>(q1, 256, 1, np, pid, pl, pc, found, far);
                }
            } else {
                const uint64_t pm = meets(lo4, np, pid, pl);
                if (W::unlikely(pm != 0)) meet<false, false>(q0, 0, lo4, pm, 0, pid, pl, pc, found, far);
                if (W::unlikely(q0.tail > 256)) meet_from<false, false>(q0, 256, 0, np, pid, pl, pc, found, far);
            }
        }
        uint32_t hend = found;       // disjoint parts that end at their sum: no gap
        uint32_t norph = 0, npromo = 0, ngated = 0;
        uint64_t hits = 0;           // met runs that are hits
        uint32_t hitS = 0, hitM = 0;
        if (W::unlikely(nm > 0)) {
            const uint64_t inl = ~0ull >> (64u - nm);
            hits = inl;
            if (found != far) {
                hend = 0;
                for (uint32_t it = 0; it < nm; ++it) {
                    const uint64_t m = W::ballot(md == hend) & inl;
                    if (!m) break;
                    hend += W::rdl(mw, W::ffs(m)) & kLen;
                }
                norph = found - hend;
                hits = W::ballot(md < hend) & inl;
                for (uint64_t om = inl & ~hits; om; om &= om - 1) {
                    const uint32_t w = W::rdl(mw, W::ffs(om));
                    res = W::mad01(is_lane(u_owner(w)), 0u - (w & kLen), res);
                }
                resident -= (int32_t)norph;
            }
            if (kPol == PS && ((q.info >> 16) & 1u) && adm) {
                // Eq. 4: proven reuse of a block of (g, c, p), not yet REUSE
                const vu mine = (mw >> kOwnS) & 255u;      // owner and contract
                const vb el = (mine == (g | (c << 6))) & (mx == q.prefix);
                const vb once = (mw & kClsM) != (kReuseCls << kClsS);
                const uint64_t em = W::ballot(el) & W::ballot(once) & hits;
                if (em) {
                    uint32_t ne = 0;
                    for (uint64_t t = em; t; t &= t - 1) ne += W::rdl(mw, W::ffs(t)) & kLen;
                    const bool open = W::rdl64(raw_debt(), (int)g) <= P.eps || (P.flags & 2);
                    if (open) {
                        npromo = ne;
                        mw = W::sel(W::of_mask(em), (mw & ~kClsM) | (kReuseCls << kClsS), mw);
                    } else {
                        ngated = ne;
                    }
                }
            }
            if (kPol == S3) {
                touch_s3(r, hits, hitS, hitM);
                load(q0, S);
                load(q1, M);
            }
        }
        const uint32_t m = nn - hend;

        // ---- reclamation
        int32_t e;
        if (kPol == SQ) e = (int32_t)m - ((int32_t)room - (int32_t)W::rdl(res, (int)g));
        else e = (int32_t)m - (P.C - resident);
        if (W::likely(e > 0)) {
            if (kPol == LRU) take(0u, 0u, -1, 0u, (uint32_t)e);
            else if (kPol == PS) evict_ps((uint32_t)e);
            else if (kPol == SQ) take(kOwnM, g << kOwnS, (int32_t)g, 0u, (uint32_t)e);
            else evict_s3((uint32_t)e, r + 1u, S, M);
            n_evc = W::mad01(me, (uint32_t)e, n_evc);
        } else {
            e = 0;
        }

        // ---- charge (Eq. 2), class of the new blocks, admission
        uint32_t nw = g << kOwnS;            // attributes of the new blocks
        const int32_t cost = -(int32_t)(m << 16);     // m <= 32,767
#pragma unroll
        for (int cc = 0; cc < kC; ++cc)
            if (kK1 || (uint32_t)cc == c) {
                E[cc] = W::mad64(me, cost, E[cc]);
                if (kPol == PS) {
                    const int64_t bal = W::rdl64(E[cc], (int)g);
                    const uint32_t cl = (bal < -P.eps || !adm) ? kProbCls : kNormalCls;
                    nw |= (c << kConS) | (cl << kClsS);
                }
            }
        res = W::mad01(me, m, res);
        resident += (int32_t)m;

        // ---- new blocks and released blocks enter the queue, deepest first
        if (kPol == S3) {
            if (m > 0) insert_s3(r, np, pid, pl, pc, hend, nw, m, ghosts || gtail > 256);
            s_unp += (int32_t)hitS;
            m_unp += (int32_t)hitM;
        } else {
            if (kQ) count_queue(me, seg_of(nw), m);
            release(np, pid, pl, pc, hend, nw, m, q.prefix, hits);
        }

        // ---- counters and the accounting of every group
        n_req = n_req + me;
        n_probe = W::mad01(me, n, n_probe);
        n_hit = W::mad01(me, hend, n_hit);
        if (W::unlikely(((nn ^ n) | (n ^ q.n_full) | norph | npromo | ngated) != 0)) {
            c_dup = c_dup + W::widen(W::mad01(me, n - nn, zu));
            c_trunc = c_trunc + W::widen(me) * (int64_t)(q.n_full - n);
            c_orph = c_orph + W::widen(W::mad01(me, norph, zu));
            c_promo = c_promo + W::widen(W::mad01(me, npromo, zu));
            c_gated = c_gated + W::widen(W::mad01(me, ngated, zu));
        }
        const vl d = raw_debt();
        d_sum = d_sum + d;
        d_max = W::vmax(d_max, d);
        res_max = W::vmax(res_max, res);
        rmax = W::vmax(rmax, wv.vu0((uint32_t)resident));
        last_h = (int32_t)hend;
        last_m = (int32_t)m;
        last_e = e;
        last_o = (int32_t)norph;
        return adm || m > 0;
    }
    // 32-bit counters into the 64-bit ones, once in kFlush requests at least
    // (a request adds at most 32,767 to each, and reinserts every block three
    // times at most).
    PC_RUNS_FN void flush() {
        c_evw = c_evw + W::widen(evw);
        c_req = c_req + W::widen(n_req);
        c_probe = c_probe + W::widen(n_probe);
        c_hit = c_hit + W::widen(n_hit);
        c_evc = c_evc + W::widen(n_evc);
        evw = n_req = n_probe = n_hit = n_evc = wv.vu0(0);
        c_moves = c_moves + W::widen(n_moves);
        c_reins = c_reins + W::widen(n_reins);
        c_ghits = c_ghits + W::widen(n_ghits);
        c_gins = c_gins + W::widen(n_gins);
        n_moves = n_reins = n_ghits = n_gins = W::hold(wv.vu0(0));
    }

    // The request's blocks enter the free queue deepest first: new blocks
    // (one run per piece), then the hits in the order of their depth.  Hits
    // that continue each other inside a piece, with equal attributes, become
    // one run again, and so do the last hit and the new blocks behind it.
    PC_RUNS_FN void release(uint32_t np, vu pid, vu pl, vu pc, uint32_t hend, uint32_t nw, uint32_t m, uint32_t p,
                            uint64_t hits) {
        const uint32_t nh = (uint32_t)W::popc(hits);
        uint32_t cd = hend;                                   // depth reached, going up
        uint32_t clo = 0, clen = 0, cat = nw, cx = p, cp = kNone;    // run being built
        // deepest piece first; the shallowest new one may continue a hit
        const vb isn = pl > 0u;
        for (uint64_t nmask = W::ballot(isn & (pc + pl > hend)); nmask;) {
            const int i = 63 - W::clz(nmask);
            nmask &= ~(1ull << i);
            const uint32_t at = W::rdl(pc, i);
            const uint32_t off = hend > at ? hend - at : 0u;
            clo = W::rdl(pid, i) + off;
            clen = W::rdl(pl, i) - off;
            cp = (uint32_t)i;
            if (nmask) push(q0, clo, clen | cat, cx);
        }
        for (uint32_t it = 0; it < nh; ++it) {
            const uint64_t mk = W::ballot(md + (mw & kLen) == cd) & hits;
            if (W::unlikely(!mk)) { over = 1; return; }        // cannot happen: the hits tile [0, hend)
            const int l = W::ffs(mk);
            const uint32_t w = W::rdl(mw, l), lo = W::rdl(mlo, l), len = w & kLen;
            const uint32_t x = kX ? W::rdl(mx, l) : 0u, i = W::rdl(mi, l);
            if (kQ) count_queue(is_lane(u_owner(w)), seg_of(w), len);
            if (i == cp && lo + len == clo && (w & kAttr) == cat && (!kX || x == cx)) {
                clo = lo;
                clen += len;
            } else {
                if (clen) push(q0, clo, clen | cat, cx);
                clo = lo;
                clen = len;
                cat = w & kAttr;
                cx = x;
                cp = i;
            }
            cd -= len;
        }
        if (clen) push(q0, clo, clen | cat, cx);
    }

    // S3-FIFO: hits stay in their queue, one access more, pinned for the
    // request; a run that is met in part becomes two, its deeper part first.
    // Orphans leave.  Runs of a window go in the order of their positions,
    // last first: a split moves only the runs behind it.
    PC_RUNS_FN void touch_s3(uint32_t r, uint64_t hits, uint32_t &hitS, uint32_t &hitM) {
        uint64_t left = ~0ull >> (64u - nm);
        while (left) {
            int k = W::ffs(left);
            if (left & (left - 1)) {
                const vu key = W::sel(W::of_mask(left), mx + 1u, wv.vu0(0));
                k = W::ffs(W::ballot(key == W::wmax(key)) & left);
            }
            left &= ~(1ull << k);
            const uint32_t at = W::rdl(mx, k), lo = W::rdl(mlo, k), ov = W::rdl(mw, k) & kLen;
            const bool hit = (hits >> k) & 1u;
            if (at & 1u) {
                m_unp -= (int32_t)ov;
                if (hit) hitM += ov;
                touch_run(q1, at >> 1, lo, ov, hit, r + 1u);
            } else {
                s_unp -= (int32_t)ov;
                if (hit) hitS += ov; else s_size -= (int32_t)ov;
                touch_run(q0, at >> 1, lo, ov, hit, r + 1u);
            }
        }
    }
    PC_RUNS_FN void touch_run(Window &rg, uint32_t pos, uint32_t lo, uint32_t ov, bool hit, uint32_t pin) {
        W::sync();
        uint32_t at = entry(pos);
        const uint32_t full = wv.ld1(rg.p + kW, at);
        const uint32_t rest = (full & kLen) - ov;
        if (W::unlikely(!hit)) {
            put2(rg, at, rest ? lo + ov : kNone, rest ? full - ov : kDead);
            return;
        }
        const uint32_t f = (full >> kFrqS) & 3u;
        const uint32_t hw = (full & kAttr & ~(3u << kFrqS)) | ((f < 3u ? f + 1u : 3u) << kFrqS) | ov;
        if (W::unlikely(rest)) {
            if (rg.tail >= W::uni(rg.cap)) { over = 1; return; }
            open_gap(rg, pos);
            put2(rg, at, lo + ov, full - ov);
            at = entry(pos + 1u);
        }
        put3(rg, at, lo, hw, pin);
    }
    // New blocks enter the small queue, or the main queue where the ghost
    // remembers them, deepest first.
    PC_RUNS_FN void insert_s3(uint32_t r, uint32_t np, vu pid, vu pl, vu pc, uint32_t hend, uint32_t nw, uint32_t m,
                              bool ghosts) {
        const vu zu = wv.vu0(0);
        const vb isn = (pl > 0u) & (pc + pl > hend);
        const vu off = W::sel(pc < hend, wv.vu0(hend) - pc, zu);
        const vu a = pid + off, L = W::sel(isn, pl - off, zu);
        nm = 0;
        uint32_t nghost = 0, far = 0;
        if (W::unlikely(ghosts && P.g_cap > 0)) meet_from<false, true>(gh, 0, 0, np, a, L, zu, nghost, far);
        uint64_t nmask = W::ballot(isn);
        uint64_t inl = 0;
        if (W::unlikely(nm > 0)) {
            if (over || q0.tail + (uint32_t)W::popc(nmask) + nm > W::uni(q0.cap) || q1.tail + nm > W::uni(q1.cap)) { over = 1; return; }
            inl = ~0ull >> (64u - nm);
        }
        while (nmask) {
            const int i = 63 - W::clz(nmask);
            nmask &= ~(1ull << i);
            const uint32_t lo = W::rdl(a, i);
            uint32_t end = lo + W::rdl(L, i);
            uint64_t gm = inl ? W::ballot(mi == (uint32_t)i) & inl : 0ull;
            while (gm) {       // the ghost's parts of this piece, deepest first
                int l = W::ffs(gm);
                if (gm & (gm - 1)) {
                    const vu key = W::sel(W::of_mask(gm), mlo - lo + 1u, zu);
                    l = W::ffs(W::ballot(key == W::wmax(key)) & gm);
                }
                gm &= ~(1ull << l);
                const uint32_t x0 = W::rdl(mlo, l), xl = W::rdl(mw, l) & kLen;
                if (x0 + xl < end) push(q0, x0 + xl, (end - x0 - xl) | nw, r);
                push(q1, x0, xl | nw, r);
                end = x0;
            }
            if (end > lo) push(q0, lo, (end - lo) | nw, r);
        }
        s_size += (int32_t)(m - nghost);
        s_unp += (int32_t)(m - nghost);
        m_unp += (int32_t)nghost;
        n_ghits = n_ghits + nghost;
    }
};

}  // namespace pcr
