// pc_runs.h -- replay of one cache instance by one wavefront, on runs of
// blocks instead of single blocks.
//
// The trace analysis (pc_intern.hip) numbers every distinct block key by the
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
// runs (30-60 for 4,096 blocks of one-touch prompts) with the attributes
// that the policies look at.  Lookup, reclamation and release then cost a
// few wavefront steps for a whole request, with no key compares, no hash
// table and no barriers.
//
// Layout of a run: its first id, and a word of length (bits 0-15) and
// attributes: owner group (16-21), contract (22-23), retention class
// (24-25), S3-FIFO frequency (26-27); PrefixShield adds the prefix id,
// S3-FIFO the request that pins it, the ghost the sequence of its last id.
// Runs live in LDS rings in free-queue order; a run emptied by hits or
// evictions stays behind with length 0 until the ring is compacted.
//
// The code is written for one wavefront with uniform control flow: `vu`,
// `vl` and `vb` are a per-lane 32-bit word, 64-bit integer and condition,
// everything else is uniform.  On the device they are the plain types; a
// host build (PC_RUNS_HOST) takes 64-lane structures instead and runs the
// same source on the CPU, lane by lane.
//
// An instance that needs more runs than its rings hold, or more pieces per
// request than lanes, is left to the general kernel (pc_replay.hip).
#pragma once
#include <stdint.h>

namespace pcr {

// One request as the trace analysis leaves it (32 bytes, read by every
// instance of the trace with scalar loads).
struct RunReq {
    uint32_t n_full;     // full blocks
    uint32_t np;         // pieces
    uint32_t info;       // bits 0-7 group, 8-15 contract, 16: its prefix was referenced before
    uint32_t prefix;
    int64_t tick;
    uint32_t ko;         // its pieces start at pieces[ko] of the trace's key buffer
    uint32_t pad;
};
// One piece: its first id, and its depth in the request (bit 31: an earlier
// piece of the request holds the same blocks -- duplicates, skipped).
struct RunPiece {
    uint32_t id, depth;
};
constexpr uint32_t kPieceDup = 0x80000000u;

// Ring entries of an instance.  Runs of fewer than 4 (small caches) or 8
// blocks on average overflow it.
constexpr int32_t runs_ring(int32_t capacity) {
    if (capacity <= 512) return 512;
    int32_t q = 1024;
    while (q * 8 < capacity) q *= 2;
    return q;
}
constexpr int kRunList = 64;     // runs of the cache that one request may meet

// LDS words of one instance.
constexpr int32_t runs_lds_bytes(int policy, int32_t q) {
    const int rings = policy == 1 ? 9 : policy == 2 ? 3 : 2;    // S3-FIFO: small, main, ghost
    return 4 * (rings * q + 5 * kRunList);
}

constexpr int kRunOk = 0, kRunGeneral = 1, kRunBroken = 2;

// Replay parameters of one instance (uniform).
struct RunParams {
    int32_t C, G, K, flags;
    int32_t s_cap, g_cap, move_thr;
    uint32_t q;                      // ring entries (a power of two)
    int64_t eps;
    int64_t rho[4], beta[4], invw[4];
    int64_t n_req;
};

// `W` supplies the lane types and wavefront operations.
template <class W, int kPol>
struct RunReplay {
    using vu = typename W::vu;
    using vl = typename W::vl;
    using vb = typename W::vb;
    using Lds = typename W::Lds;
    static constexpr int LRU = 0, S3 = 1, PS = 2, SQ = 3;
    static constexpr uint32_t kLen = 0xFFFFu, kAttr = 0xFFFF0000u;
    static constexpr int kOwnS = 16, kConS = 22, kClsS = 24, kFrqS = 26;
    static constexpr uint32_t kReuseCls = 2, kNormalCls = 1, kProbCls = 0;
    static constexpr uint32_t kNone = 0xFFFFFFFFu;

    struct Ring {
        Lds lo, w, x;
        uint32_t head, tail;
        uint32_t lim;            // compact when the window would grow past this
    };

    const RunParams &P;
    W &wv;
    const vu lane;
    const uint32_t qm;           // ring index mask
    Ring q0, q1, gh;             // free queue (S3-FIFO: small, main, ghost)
    Lds xd, xlo, xw, xx, xi;     // the runs the current request meets
    bool general;                // leave the instance to the general kernel

    // uniform state
    int32_t resident, rmax;
    int32_t s_size, s_unp, m_unp;
    uint32_t gseq;
    uint64_t ev_total, s3_moves, s3_reins, s3_ghits, s3_gins;
    int64_t tprev;
    int32_t last_h, last_m, last_e, last_o;
    // lane x = group x
    vl E[4];                     // effective balances at tprev (Eq. 1)
    vl d_max, d_sum;
    vu cnt0, cnt1, cnt2;         // queued blocks per segment (PrefixShield, StaticQuota: cnt0)
    vu res, res_max;
    vl evw, c_probe, c_hit, c_dup, c_trunc, c_promo, c_gated, c_orph, c_evc, c_req;

    static PC_RUNS_FN uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }

    PC_RUNS_FN RunReplay(const RunParams &p, W &w, Lds base) : P(p), wv(w), lane(w.lane()), qm(p.q - 1u) {
        Lds at = base;
        auto ring = [&](Ring &r, bool x) {
            r.lo = at; at = at + P.q;
            r.w = at; at = at + P.q;
            r.x = at;
            if (x) at = at + P.q;
            r.head = r.tail = 0;
            r.lim = 64;
        };
        ring(q0, kPol == S3 || kPol == PS);
        if (kPol == S3) { ring(q1, true); ring(gh, true); }
        xd = at; at = at + kRunList;
        xlo = at; at = at + kRunList;
        xw = at; at = at + kRunList;
        xx = at; at = at + kRunList;
        xi = at;
        general = false;
        resident = rmax = 0;
        s_size = s_unp = m_unp = 0;
        gseq = 0;
        ev_total = s3_moves = s3_reins = s3_ghits = s3_gins = 0;
        tprev = 0;
        last_h = last_m = last_e = last_o = 0;
        const vl z = wv.vl0(0);
        const vu zu = wv.vu0(0);
        for (int c = 0; c < 4; ++c) E[c] = wv.vl0(c < P.K ? P.beta[c] : 0);
        d_max = d_sum = z;
        cnt0 = cnt1 = cnt2 = res = res_max = zu;
        evw = c_probe = c_hit = c_dup = c_trunc = c_promo = c_gated = c_orph = c_evc = c_req = z;
    }

    // ------------------------------------------------------------ debts
    // Eqs. 1 and 3: balances move to tick t.  The lazy refill of Eq. 1
    // composes exactly: min(beta, min(beta, B + rho d1) + rho d2) =
    // min(beta, B + rho (d1 + d2)), so the balances are kept at the last
    // tick and every request adds one uniform amount.  2^62 stands for any
    // amount that certainly reaches beta (balances stay above -2^61).
    PC_RUNS_FN void refill(int64_t t) {
        const uint64_t dt = (uint64_t)(t - tprev);
        tprev = t;
        if (dt == 0) return;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (c < P.K) {
                uint64_t inc = (uint64_t)P.rho[c] * dt;
                if (W::mulhi((uint64_t)P.rho[c], dt) != 0 || inc > (1ull << 62)) inc = 1ull << 62;
                E[c] = W::vmin(E[c] + (int64_t)inc, P.beta[c]);
            }
    }
    PC_RUNS_FN vl raw_debt() const {
        vl d = W::vmax(-E[0], (int64_t)0);
        if (P.K > 1)
#pragma unroll
            for (int c = 1; c < 4; ++c)
                if (c < P.K) d = d + W::vmax(-E[c], (int64_t)0);
        return d;
    }
    // Eq. 5 (1/w_c in Q16) and Eq. 8's decrement
    PC_RUNS_FN void norm_debt(vl &d, vl &dec) const {
        if (P.K == 1) {     // w = 1
            d = W::vmax(-E[0], (int64_t)0);
            dec = W::sel(E[0] < (int64_t)0, wv.vl0(65536), wv.vl0(0));
            return;
        }
        d = wv.vl0(0);
        dec = wv.vl0(0);
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (c < P.K) {
                const vb neg = E[c] < (int64_t)0;
                d = d + W::sel(neg, W::mul_shr16(-E[c], P.invw[c]), wv.vl0(0));
                const vb take = neg & ((dec == (int64_t)0) | (wv.vl0(P.invw[c]) < dec));
                dec = W::sel(take, wv.vl0(P.invw[c]), dec);
            }
    }

    // ------------------------------------------------------------ rings
    PC_RUNS_FN static vu owner(vu w) { return (w >> kOwnS) & 63u; }
    PC_RUNS_FN static vu cls(vu w) { return (w >> kClsS) & 3u; }
    PC_RUNS_FN static uint32_t u_owner(uint32_t w) { return (w >> kOwnS) & 63u; }
    PC_RUNS_FN static uint32_t u_cls(uint32_t w) { return (w >> kClsS) & 3u; }

    // Live runs move to the front of the window, in order.
    template <bool kX>
    PC_RUNS_FN void compact(Ring &r) {
        uint32_t nw = r.head;
        for (uint32_t b = r.head; b < r.tail; b += 64) {
            W::sync();
            const vu pos = lane + b;
            const vu at = pos & qm;
            const vu lo = W::ld(r.lo, at), w = W::ld(r.w, at);
            vu x = w;
            if (kX) x = W::ld(r.x, at);
            const vb live = (pos < r.tail) & ((w & kLen) > 0u);
            const uint64_t lm = W::ballot(live);
            const vu to = (W::mbcnt(lm) + nw) & qm;
            W::st(live, r.lo, to, lo);
            W::st(live, r.w, to, w);
            if (kX) W::st(live, r.x, to, x);
            nw += (uint32_t)W::popc(lm);
        }
        const uint32_t live = nw - r.head;
        r.head &= qm;            // (positions stay far below 2^32)
        r.tail = r.head + live;
        uint32_t lim = (live + live / 2 + 95u) & ~63u;
        r.lim = umin(lim, P.q);
    }
    // Room for k more entries (the window never exceeds the ring).
    template <bool kX>
    PC_RUNS_FN bool room_for(Ring &r, uint32_t k) {
        if (r.tail + k - r.head <= r.lim) return true;
        compact<kX>(r);
        const uint32_t need = r.tail + k - r.head;
        if (need > P.q) { general = true; return false; }
        if (need > r.lim) r.lim = umin((need + 63u) & ~63u, P.q);
        return true;
    }
    PC_RUNS_FN void push(Ring &r, uint32_t lo, uint32_t w, uint32_t x, bool has_x) {
        const uint32_t at = r.tail & qm;
        wv.st1(r.lo, at, lo);
        wv.st1(r.w, at, w);
        if (has_x) wv.st1(r.x, at, x);
        r.tail += 1;
    }
    // The run at window position `pos` becomes two: everything from pos + 1
    // on moves up by one entry.
    PC_RUNS_FN void open_gap(Ring &r, uint32_t pos) {
        const uint32_t first = pos + 1;
        uint32_t e = r.tail;
        while (e > first) {
            const uint32_t b = e - first > 64u ? e - 64u : first;
            W::sync();
            const vu p = lane + b;
            const vb in = p < e;
            const vu from = p & qm, to = (p + 1u) & qm;
            const vu lo = W::ld(r.lo, from), w = W::ld(r.w, from), x = W::ld(r.x, from);
            W::st(in, r.lo, to, lo);
            W::st(in, r.w, to, w);
            W::st(in, r.x, to, x);
            e = b;
        }
        r.tail += 1;
    }

    // Evicted blocks, `take` of them from each lane's run of word w.
    PC_RUNS_FN void count_evicted(vu w, vu take) {
        uint64_t vm = W::ballot(take > 0u);
        while (vm) {
            const int l = W::ffs(vm);
            vm &= vm - 1;
            const uint32_t o = u_owner(W::rdl(w, l)), n = W::rdl(take, l);
            const vb me = lane == o;
            evw = evw + W::widen(W::sel(me, wv.vu0(n), wv.vu0(0)));
            res = res - W::sel(me, wv.vu0(n), wv.vu0(0));
        }
    }
    // One queue count per (owner, segment): d blocks more or fewer.
    PC_RUNS_FN void count_queue(uint32_t o, uint32_t seg, uint32_t d) {
        const vu dv = W::sel(lane == o, wv.vu0(d), wv.vu0(0));
        if (seg == 0) cnt0 = cnt0 + dv;
        else if (seg == 1) cnt1 = cnt1 + dv;
        else cnt2 = cnt2 + dv;
    }
    PC_RUNS_FN uint32_t seg_of(uint32_t w) const {
        return (kPol == PS && !(P.flags & 1)) ? u_cls(w) : 0u;
    }

    // k victims from the queue, oldest first: only blocks owned by x (x >= 0)
    // of segment s (s >= 0).
    PC_RUNS_FN void take(int32_t x, int32_t s, uint32_t k) {
        uint32_t rem = k;
        W::sync();
        for (uint32_t b = q0.head; b < q0.tail && rem > 0; b += 64) {
            const vu pos = lane + b;
            const vu at = pos & qm;
            const vu w = W::ld(q0.w, at);
            vb ok = pos < q0.tail;
            if (kPol != LRU && x >= 0) ok = ok & (owner(w) == (uint32_t)x);
            if (kPol == PS && s >= 0) ok = ok & (cls(w) == (uint32_t)s);
            const vu len = W::sel(ok, w & kLen, wv.vu0(0));
            if (W::ballot(len > 0u) == 0) continue;
            const vu upto = W::scan(len);
            const vu before = upto - len;
            const vu tk = W::sel(before < rem, W::vmin(len, wv.vu0(rem) - before), wv.vu0(0));
            const uint32_t tot = W::rdl(upto, 63);
            const uint32_t nv = umin(tot, rem);
            W::st(tk > 0u, q0.w, at, w - tk);
            count_evicted(w, tk);
            if (kPol == PS || kPol == SQ) {
                uint64_t vm = W::ballot(tk > 0u);
                while (vm) {
                    const int l = W::ffs(vm);
                    vm &= vm - 1;
                    const uint32_t wl = W::rdl(w, l);
                    count_queue(u_owner(wl), seg_of(wl), 0u - W::rdl(tk, l));
                }
            }
            rem -= nv;
            resident -= (int32_t)nv;
            ev_total += nv;
        }
        if (rem) general = true;    // cannot happen: the counts say that the queue holds k
    }
    // Window position of the oldest live run of (x, s).
    PC_RUNS_FN uint32_t head_pos(uint32_t x, int32_t s) const {
        W::sync();
        for (uint32_t b = q0.head; b < q0.tail; b += 64) {
            const vu pos = lane + b;
            const vu w = W::ld(q0.w, pos & qm);
            vb ok = (pos < q0.tail) & ((w & kLen) > 0u) & (owner(w) == x);
            if (s >= 0) ok = ok & (cls(w) == (uint32_t)s);
            const uint64_t m = W::ballot(ok);
            if (m) return b + (uint32_t)W::ffs(m);
        }
        return kNone;
    }
    // Alg. 2 (Eqs. 5-9): runs of victims from the group with the largest
    // projected debt.
    PC_RUNS_FN void evict_ps(uint32_t e) {
        const int nseg = (P.flags & 1) ? 1 : 3;
        const vb grp = lane < (uint32_t)P.G;
        vl Pd, D;
        norm_debt(Pd, D);
        vu avail = cnt0 + cnt1 + cnt2;
        uint32_t rem = e;
        while (rem > 0 && !general) {
            const vb inE = grp & (avail > 0u) & (Pd > P.eps);          // Eq. 6
            const uint64_t Em = W::ballot(inE);
            if (!Em) break;
            int gs;
            int64_t pg, thr = P.eps;
            if ((Em & (Em - 1)) == 0) {      // one indebted candidate owner
                gs = W::ffs(Em);
                pg = W::rdl64(Pd, gs);
            } else {
                pg = W::wmax64(W::sel(inE, Pd, wv.vl0(-1)));           // Eq. 7
                uint64_t tied = W::ballot(inE & (Pd == pg));
                gs = W::ffs(tied);
                if (tied & (tied - 1)) {     // ties: lowest non-empty segment, then the oldest head
                    const vu seg = W::sel(cnt0 > 0u, wv.vu0(0), W::sel(cnt1 > 0u, wv.vu0(1), wv.vu0(2)));
                    int mseg = nseg == 1 ? 0 : 2;
                    if (nseg == 3) {
                        for (int s = 1; s >= 0; --s)
                            if (W::ballot(seg == (uint32_t)s) & tied) mseg = s;
                        tied &= W::ballot(seg == (uint32_t)mseg);
                        gs = W::ffs(tied);
                    }
                    if (tied & (tied - 1)) {
                        uint32_t best = kNone;
                        for (uint64_t tm = tied; tm; tm &= tm - 1) {
                            const int x = W::ffs(tm);
                            const uint32_t hp = head_pos((uint32_t)x, nseg == 1 ? -1 : mseg);
                            if (hp < best) { best = hp; gs = x; }
                        }
                    }
                }
                const int64_t p2 = W::wmax64(W::sel(inE & (lane != (uint32_t)gs), Pd, wv.vl0(-1)));
                if (p2 > thr) thr = p2;
            }
            const int64_t dg = W::rdl64(D, gs);
            if (dg <= 0) { general = true; break; }    // cannot happen: an indebted group has a decrement
            const uint32_t ag = W::rdl(avail, gs);
            // the group keeps winning strictly while P - i D > max(second, eps)
            uint64_t k = 1;
            if (pg > thr) {
                const uint64_t num = (uint64_t)(pg - thr) + (uint64_t)dg - 1;
                k = P.K == 1 ? num >> 16 : W::udiv(num, (uint64_t)dg);
                if (k < 1) k = 1;
            }
            if (k > rem) k = rem;
            if (k > ag) k = ag;
            uint32_t kk = (uint32_t)k;
            if (nseg == 1) {
                take(gs, -1, kk);
            } else {
                for (int s = 0; s < 3 && kk > 0; ++s) {
                    const uint32_t cs = W::rdl(s == 0 ? cnt0 : s == 1 ? cnt1 : cnt2, gs);
                    const uint32_t tk = umin(cs, kk);
                    if (tk > 0) take(gs, s, tk);
                    kk -= tk;
                }
            }
            const vb me = lane == (uint32_t)gs;
            const vl np = Pd - (int64_t)k * dg;
            Pd = W::sel(me, W::vmax(np, (int64_t)0), Pd);
            avail = W::sel(me, avail - (uint32_t)k, avail);
            rem -= (uint32_t)k;
        }
        // no indebted candidate owner: global segment order (Eq. 9 fallback)
        for (int s = 0; s < nseg && rem > 0 && !general; ++s) {
            const uint32_t tot = W::wsum(s == 0 ? cnt0 : s == 1 ? cnt1 : cnt2);
            const uint32_t tk = umin(tot, rem);
            if (tk > 0) take(-1, nseg == 1 ? -1 : s, tk);
            rem -= tk;
        }
        if (rem > 0) general = true;
    }

    // ------------------------------------------------------------ S3-FIFO
    // Position of the oldest live run that the request does not pin.
    PC_RUNS_FN uint32_t first_unpinned(Ring &r, uint32_t pin, uint32_t &lo, uint32_t &w) {
        W::sync();
        for (uint32_t b = r.head; b < r.tail; b += 64) {
            const vu pos = lane + b;
            const vu at = pos & qm;
            const vu wl = W::ld(r.w, at), ll = W::ld(r.lo, at), xl = W::ld(r.x, at);
            const vb live = (pos < r.tail) & ((wl & kLen) > 0u);
            if (b == r.head) {     // runs emptied at the front leave the window
                const uint64_t lm = W::ballot(live);
                if (!lm) { r.head = umin(b + 64, r.tail); continue; }
                r.head += (uint32_t)W::ffs(lm);
            }
            const uint64_t m = W::ballot(live & (xl != pin));
            if (m) {
                const int l = W::ffs(m);
                lo = W::rdl(ll, l);
                w = W::rdl(wl, l);
                return b + (uint32_t)l;
            }
        }
        return kNone;
    }
    PC_RUNS_FN void evict_s3(uint32_t e, uint32_t pin) {
        uint32_t rem = e;
        while (rem > 0 && !general) {
            const bool useS = (s_size >= P.s_cap && s_unp > 0) || m_unp == 0;
            uint32_t lo = 0, w = 0;
            if (useS) {
                const uint32_t pos = first_unpinned(q0, pin, lo, w);
                if (pos == kNone) { general = true; break; }
                // how many of the run's blocks (deepest first) go before the
                // one-at-a-time rule would look at the main queue
                const uint32_t len = w & kLen;
                const int32_t la = s_size - P.s_cap + 1 < s_unp ? s_size - P.s_cap + 1 : s_unp;
                uint32_t k;
                if ((int32_t)((w >> kFrqS) & 3u) >= P.move_thr) {
                    // (the first move gives the main queue an unpinned block)
                    k = umin(len, m_unp == 0 ? (la > 1 ? (uint32_t)la : 1u) : (uint32_t)la);
                    wv.st1(q0.w, pos & qm, w - k);
                    if (!room_for<true>(q1, 1)) break;
                    push(q1, lo + len - k, k | (w & kAttr & ~(3u << kFrqS)), pin - 1u, true);
                    s3_moves += k;
                    m_unp += (int32_t)k;
                } else {
                    k = umin(len, rem);
                    if (m_unp > 0) k = umin(k, (uint32_t)la);
                    wv.st1(q0.w, pos & qm, w - k);
                    victims(w, k);
                    if (P.g_cap > 0) {
                        if (!ghost_room()) break;
                        push(gh, lo + len - k, k, gseq, true);
                    }
                    gseq += k;
                    s3_gins += k;
                    rem -= k;
                }
                s_size -= (int32_t)k;
                s_unp -= (int32_t)k;
            } else {
                const uint32_t pos = first_unpinned(q1, pin, lo, w);
                if (pos == kNone) { general = true; break; }
                const uint32_t len = w & kLen;
                if ((w >> kFrqS) & 3u) {
                    wv.st1(q1.w, pos & qm, w - len);
                    if (!room_for<true>(q1, 1)) break;
                    push(q1, lo, w - (1u << kFrqS), pin - 1u, true);
                    s3_reins += len;
                } else {
                    const uint32_t k = umin(umin(len, rem), (uint32_t)m_unp);
                    wv.st1(q1.w, pos & qm, w - k);
                    victims(w, k);
                    m_unp -= (int32_t)k;
                    rem -= k;
                }
            }
        }
    }
    PC_RUNS_FN void victims(uint32_t w, uint32_t k) {
        const vu d = W::sel(lane == u_owner(w), wv.vu0(k), wv.vu0(0));
        evw = evw + W::widen(d);
        res = res - d;
        resident -= (int32_t)k;
        ev_total += k;
    }
    // Ids of a ghost run that have left the window of the last g_cap
    // insertions (its deepest ids went in first).
    PC_RUNS_FN vu expired(vu w, vu base) const {
        const vu age = wv.vu0(gseq - (uint32_t)P.g_cap) - base;     // signed
        const vu len = w & kLen;
        return W::sel((age >> 31) > 0u, wv.vu0(0), W::vmin(age, len));
    }
    // Room for one more ghost run: runs that left the window are dropped
    // where they are first in the ring, and all of them by a compaction.
    PC_RUNS_FN bool ghost_room() {
        if (gh.tail + 1 - gh.head <= gh.lim) return true;
        W::sync();
        for (uint32_t b = gh.head; b < gh.tail; b += 64) {
            const vu pos = lane + b;
            const vu at = pos & qm;
            const vu w = W::ld(gh.w, at), base = W::ld(gh.x, at);
            const vu ex = expired(w, base);
            const vb in = (pos < gh.tail) & (ex > 0u);
            W::st(in, gh.w, at, w - ex);
            W::st(in, gh.x, at, base + ex);
        }
        return room_for<true>(gh, 1);
    }

    // ------------------------------------------------------------ lookup
    // Runs of ring r that the request's pieces [pa, pa + pl) meet: their
    // leading part is filed in the list with its depth in the request, and
    // taken off the run (kKeep: left there, its window position filed).  By
    // (a) at the top a run meets one piece at most.
    template <bool kX, bool kKeep, bool kGhost>
    PC_RUNS_FN uint32_t match(Ring &r, uint32_t nm, uint32_t ringbit, uint32_t np, vu pa, vu pl, vu pc) {
        W::sync();
        for (uint32_t b = r.head; b < r.tail; b += 64) {
            const vu pos = lane + b;
            const vu at = pos & qm;
            vu lo = W::ld(r.lo, at), w = W::ld(r.w, at);
            vu x = w;
            if (kX) x = W::ld(r.x, at);
            const vb in = pos < r.tail;
            vu len = W::sel(in, w & kLen, wv.vu0(0));
            if (kGhost) {
                const vu ex = expired(w, x);
                len = len - W::sel(in, ex, wv.vu0(0));
            } else if (!kKeep && b == r.head) {
                const uint64_t lm = W::ballot(len > 0u);
                r.head = lm ? r.head + (uint32_t)W::ffs(lm) : umin(b + 64, r.tail);
            }
            bool any = false;
            for (uint32_t i = 0; i < np; ++i) {
                const uint32_t a = W::rdl(pa, (int)i), L = W::rdl(pl, (int)i);
                const vb m = ((lo - a) < L) & (len > 0u);
                const uint64_t mm = W::ballot(m);
                if (mm == 0) continue;
                any = true;
                const vu ov = W::vmin(len, wv.vu0(a + L) - lo);
                const vu k = W::mbcnt(mm) + nm;
                const vb ok = m & (k < (uint32_t)kRunList);
                W::st(ok, xd, k, lo - a + W::rdl(pc, (int)i));
                W::st(ok, xlo, k, lo);
                W::st(ok, xw, k, (w & kAttr) | ov);
                if (kX && !kKeep && !kGhost) W::st(ok, xx, k, x);
                if (kKeep) W::st(ok, xx, k, (pos << 1) | ringbit);
                W::st(ok, xi, k, wv.vu0(i));
                nm += (uint32_t)W::popc(mm);
                if (!kKeep) {
                    lo = W::sel(m, lo + ov, lo);
                    w = W::sel(m, w - ov, w);
                }
                len = W::sel(m, kKeep ? wv.vu0(0) : len - ov, len);
            }
            if (!kKeep && any) {
                W::st(in, r.lo, at, lo);
                W::st(in, r.w, at, w);
            }
        }
        if (nm > (uint32_t)kRunList) general = true;
        return nm;
    }

    // ------------------------------------------------------------ request
    // `pid`, `pdepth`: the request's pieces, lane i piece i (i < np <= 64).
    // `adm`: its prefix was admitted before; returns whether it is now.
    PC_RUNS_FN bool request(uint32_t r, const RunReq &q, vu pid, vu pdepth, bool adm) {
        const uint32_t g = q.info & 0xFFu, c = (q.info >> 8) & 0xFFu;
        const bool q1bit = ((q.info >> 16) & 1u) != 0;
        const uint32_t np = q.np;
        if (np > 64u || c >= (uint32_t)P.K) { general = true; return adm; }
        refill(q.tick);
        const uint32_t room = (uint32_t)(kPol == SQ ? P.C / P.G : P.C);
        const uint32_t n = umin(q.n_full, room);
        const vb me = lane == g;
        const vu zu = wv.vu0(0);

        // pieces cut to n blocks; their depths without the duplicates
        vu pl, pc;
        uint32_t nn = n;             // blocks that are no duplicates
        if (np <= 1u) {
            pl = W::sel(lane < np, wv.vu0(n), zu);
            pc = zu;
        } else {
            const vu d = pdepth & ~kPieceDup;
            const vu nx = W::sel(lane == np - 1u, wv.vu0(n), W::vmin(W::next_lane(d), wv.vu0(n)));
            pl = W::sel((lane < np) & (d < nx) & (pdepth < kPieceDup), nx - d, zu);
            const vu upto = W::scan(pl);
            pc = upto - pl;
            nn = W::rdl(upto, 63);
        }

        // ---- lookup
        uint32_t nm;
        if (kPol == S3) {
            nm = match<false, true, false>(q0, 0, 0, np, pid, pl, pc);
            nm = match<false, true, false>(q1, nm, 1, np, pid, pl, pc);
        } else {
            nm = match<kPol == PS, false, false>(q0, 0, 0, np, pid, pl, pc);
        }
        if (general) return adm;
        uint32_t hend = 0, norph = 0, npromo = 0, ngated = 0;
        vu md = zu, mlo = zu, mw = zu, mx = zu, mi = zu;
        uint64_t left = 0;           // met runs that are hits
        if (nm > 0) {
            W::sync();
            md = W::ld(xd, lane & 63u);
            mlo = W::ld(xlo, lane & 63u);
            mw = W::ld(xw, lane & 63u);
            if (kPol == PS || kPol == S3) mx = W::ld(xx, lane & 63u);
            mi = W::ld(xi, lane & 63u);
            const vb inl = lane < nm;
            md = W::sel(inl, md, zu);
            mw = W::sel(inl, mw, zu);
            const vu ml = mw & kLen;
            uint32_t found, far;
            if (nm == 1) {
                found = W::rdl(ml, 0);
                far = W::rdl(md, 0) + found;
            } else {
                found = W::wsum(ml);
                far = W::wmax(md + ml);
            }
            if (found == far) hend = found;      // disjoint parts that end at their sum: no gap
            else
                for (uint32_t it = 0; it < nm; ++it) {
                    const uint64_t m = W::ballot(inl & (md == hend));
                    if (!m) break;
                    hend += W::rdl(ml, W::ffs(m));
                }
            norph = found - hend;
            left = W::ballot(inl & (md < hend));
            const uint64_t orph = W::ballot(inl) & ~left;
            if (kPol == PS || kPol == SQ)        // hits and orphans leave their queue
                for (uint32_t k = 0; k < nm; ++k) {
                    const uint32_t w = W::rdl(mw, (int)k);
                    count_queue(u_owner(w), seg_of(w), 0u - (w & kLen));
                }
            for (uint64_t om = orph; om; om &= om - 1) {
                const uint32_t w = W::rdl(mw, W::ffs(om));
                res = res - W::sel(lane == u_owner(w), wv.vu0(w & kLen), zu);
            }
            resident -= (int32_t)norph;
            if (kPol == PS && q1bit && adm) {
                // Eq. 4: proven reuse of a block of (g, c, p), not yet REUSE
                const vb el = inl & (md < hend) & (owner(mw) == g) & (((mw >> kConS) & 3u) == c) &
                              (cls(mw) != kReuseCls) & (mx == q.prefix);
                const uint64_t em = W::ballot(el);
                if (em) {
                    const uint32_t ne = W::wsum(W::sel(el, ml, zu));
                    const bool open = W::rdl64(raw_debt(), (int)g) <= P.eps || (P.flags & 2);
                    if (open) {
                        npromo = ne;
                        mw = W::sel(el, (mw & ~(3u << kClsS)) | (kReuseCls << kClsS), mw);
                    } else {
                        ngated = ne;
                    }
                }
            }
        }
        const uint32_t m = nn - hend;
        uint32_t hitS = 0, hitM = 0;
        if (kPol == S3) touch_s3(r, nm, left, mlo, mw, mx, hitS, hitM);
        if (general) return adm;

        // ---- reclamation
        int32_t e;
        if (kPol == SQ) e = (int32_t)m - ((int32_t)room - (int32_t)W::rdl(res, (int)g));
        else e = (int32_t)m - (P.C - resident);
        if (e < 0) e = 0;
        if (e > 0) {
            if (kPol == LRU) take(-1, -1, (uint32_t)e);
            else if (kPol == PS) evict_ps((uint32_t)e);
            else if (kPol == SQ) take((int32_t)g, -1, (uint32_t)e);
            else evict_s3((uint32_t)e, r + 1u);
            if (general) return adm;
            c_evc = c_evc + W::widen(W::sel(me, wv.vu0((uint32_t)e), zu));
        }

        // ---- charge (Eq. 2), class of the new blocks, admission
        uint32_t nw = g << kOwnS;            // attributes of the new blocks
        bool adm_now = adm;
        if (m > 0) {
            const int64_t cost = (int64_t)m * 65536;
            int64_t B = 0;
#pragma unroll
            for (int cc = 0; cc < 4; ++cc)
                if (cc < P.K && (uint32_t)cc == c) {
                    E[cc] = W::sel(me, E[cc] - cost, E[cc]);
                    if (kPol == PS) B = W::rdl64(E[cc], (int)g);
                }
            if (kPol == PS) {
                const uint32_t cl = (B < -P.eps || !adm) ? kProbCls : kNormalCls;
                nw |= (c << kConS) | (cl << kClsS);
            }
            adm_now = true;
            res = res + W::sel(me, wv.vu0(m), zu);
            resident += (int32_t)m;
        }

        // ---- new blocks and released blocks enter the queue, deepest first
        if (kPol == S3) {
            if (m > 0) insert_s3(r, np, pid, pl, pc, hend, nw, m);
            s_unp += (int32_t)hitS;
            m_unp += (int32_t)hitM;
        } else {
            release(np, pid, pl, pc, hend, nw, m, q.prefix, left, md, mlo, mw, mx, mi);
        }
        if (general) return adm;

        // ---- counters and the accounting of every group
        c_req = c_req + W::widen(W::sel(me, wv.vu0(1), zu));
        c_probe = c_probe + W::widen(W::sel(me, wv.vu0(n), zu));
        c_hit = c_hit + W::widen(W::sel(me, wv.vu0(hend), zu));
        if (nn != n) c_dup = c_dup + W::widen(W::sel(me, wv.vu0(n - nn), zu));
        if (n != q.n_full) c_trunc = c_trunc + W::widen(W::sel(me, wv.vu0(q.n_full - n), zu));
        if (norph) c_orph = c_orph + W::widen(W::sel(me, wv.vu0(norph), zu));
        if (npromo) c_promo = c_promo + W::widen(W::sel(me, wv.vu0(npromo), zu));
        if (ngated) c_gated = c_gated + W::widen(W::sel(me, wv.vu0(ngated), zu));
        const vl d = raw_debt();
        d_sum = d_sum + d;
        d_max = W::vmax(d_max, d);
        res_max = W::vmax(res_max, res);
        if (resident > rmax) rmax = resident;
        last_h = (int32_t)hend;
        last_m = (int32_t)m;
        last_e = e;
        last_o = (int32_t)norph;
        return adm_now;
    }

    // The request's blocks enter the free queue deepest first: new blocks
    // (one run per piece), then the hits in the order of their depth.  Hits
    // that continue each other inside a piece, with equal attributes, become
    // one run again, and so do the last hit and the new blocks behind it.
    PC_RUNS_FN void release(uint32_t np, vu pid, vu pl, vu pc, uint32_t hend, uint32_t nw, uint32_t m, uint32_t p,
                            uint64_t hits, vu md, vu mlo, vu mw, vu mx, vu mi) {
        const uint32_t nh = (uint32_t)W::popc(hits);
        constexpr bool kX = kPol == PS;
        if (!room_for<kX>(q0, np + nh)) return;
        uint32_t cd = hend;                                   // depth reached, going up
        uint32_t clo = 0, clen = 0, cat = 0, cx = 0, cp = kNone;    // run being built
        if (m > 0) {
            const vb isn = (pl > 0u) & (pc + pl > hend);
            const uint64_t nmask = W::ballot(isn);
            // the shallowest new piece may continue a hit; the others are whole
            const int sh = W::ffs(nmask);
            const uint64_t deep = nmask & (nmask - 1);
            if (deep) {
                const uint32_t nd = (uint32_t)W::popc(deep);
                const vu at = (wv.vu0(q0.tail + nd - 1u) - W::mbcnt(deep)) & qm;
                const vb isd = isn & (lane > (uint32_t)sh);
                W::st(isd, q0.lo, at, pid);
                W::st(isd, q0.w, at, pl | nw);
                if (kX) W::st(isd, q0.x, at, wv.vu0(p));
                q0.tail += nd;
            }
            const uint32_t spc = W::rdl(pc, sh), spl = W::rdl(pl, sh);
            const uint32_t off = hend > spc ? hend - spc : 0u;
            clo = W::rdl(pid, sh) + off;
            clen = spl - off;
            cat = nw;
            cx = p;
            cp = (uint32_t)sh;
            if (kPol == PS || kPol == SQ) count_queue(u_owner(nw), seg_of(nw), m);
        }
        for (uint32_t it = 0; it < nh; ++it) {
            const uint64_t mk = W::ballot(md + (mw & kLen) == cd) & hits;
            if (!mk) { general = true; return; }    // cannot happen: the hits tile [0, hend)
            const int l = W::ffs(mk);
            const uint32_t w = W::rdl(mw, l), lo = W::rdl(mlo, l), len = w & kLen;
            const uint32_t x = kX ? W::rdl(mx, l) : 0u, i = W::rdl(mi, l);
            if (kPol == PS || kPol == SQ) count_queue(u_owner(w), seg_of(w), len);
            if (i == cp && lo + len == clo && (w & kAttr) == cat && x == cx) {
                clo = lo;
                clen += len;
            } else {
                if (clen) push(q0, clo, clen | cat, cx, kX);
                clo = lo;
                clen = len;
                cat = w & kAttr;
                cx = x;
                cp = i;
            }
            cd -= len;
        }
        if (clen) push(q0, clo, clen | cat, cx, kX);
    }

    // S3-FIFO: hits stay in their queue, one access more, pinned for the
    // request; a run that is met in part becomes two, its deeper part first.
    // Orphans leave.
    PC_RUNS_FN void touch_s3(uint32_t r, uint32_t nm, uint64_t hits, vu mlo, vu mw, vu mx, uint32_t &hitS,
                             uint32_t &hitM) {
        if (nm == 0) return;
        const vu zu = wv.vu0(0);
        const vb inl = lane < nm, isM = (mx & 1u) > 0u, isH = W::of_mask(hits);
        const vu at = (mx >> 1) & qm, ov = mw & kLen;
        const vu full = W::sel(isM, W::ld(q1.w, at), W::ld(q0.w, at));
        const vu rest = (full & kLen) - ov;
        const vu f = (full >> kFrqS) & 3u;
        const vu hw = (full & (kAttr & ~(3u << kFrqS))) | (W::vmin(f + 1u, wv.vu0(3)) << kFrqS) | ov;
        const vb whole = inl & isH & (rest == 0u), orph = inl & (!isH);
        touch_ring(q0, (!isM) & whole, (!isM) & orph, at, hw, mlo + ov, (full & kAttr) | rest, r + 1u);
        touch_ring(q1, isM & whole, isM & orph, at, hw, mlo + ov, (full & kAttr) | rest, r + 1u);
        const uint32_t all = W::wsum(W::sel(inl & isH, ov, zu));
        hitM = W::wsum(W::sel(inl & isH & isM, ov, zu));
        hitS = all - hitM;
        s_unp -= (int32_t)hitS;
        m_unp -= (int32_t)hitM;
        if (W::ballot(orph)) {
            const uint32_t oM = W::wsum(W::sel(orph & isM, ov, zu)), oS = W::wsum(W::sel(orph & (!isM), ov, zu));
            s_size -= (int32_t)oS;
            s_unp -= (int32_t)oS;
            m_unp -= (int32_t)oM;
        }
        // runs met in part, last window position first: a split moves only
        // the runs behind it
        uint64_t part = W::ballot(inl & isH & (rest > 0u));
        while (part) {
            const vu key = W::sel(W::of_mask(part), (mx >> 1) + 1u, zu);
            const uint64_t tm = W::ballot(key == W::wmax(key)) & part;
            const int k = W::ffs(tm);
            part &= ~(1ull << k);
            const uint32_t pos = W::rdl(mx, k) >> 1, lo = W::rdl(mlo, k), o = W::rdl(ov, k);
            const uint32_t dw = W::rdl(full, k) - o, tw = W::rdl(hw, k);
            if (W::rdl(mx, k) & 1u) split(q1, pos, lo, o, dw, tw, r + 1u);
            else split(q0, pos, lo, o, dw, tw, r + 1u);
        }
    }
    PC_RUNS_FN void touch_ring(Ring &rg, vb whole, vb orph, vu at, vu hw, vu olo, vu ow, uint32_t pin) {
        W::st(whole, rg.w, at, hw);
        W::st(whole, rg.x, at, wv.vu0(pin));
        W::st(orph, rg.lo, at, olo);
        W::st(orph, rg.w, at, ow);
    }
    PC_RUNS_FN void split(Ring &rg, uint32_t pos, uint32_t lo, uint32_t o, uint32_t dw, uint32_t tw, uint32_t pin) {
        if (rg.tail + 1u - rg.head > P.q) { general = true; return; }
        open_gap(rg, pos);
        wv.st1(rg.lo, pos & qm, lo + o);
        wv.st1(rg.w, pos & qm, dw);
        wv.st1(rg.lo, (pos + 1u) & qm, lo);
        wv.st1(rg.w, (pos + 1u) & qm, tw);
        wv.st1(rg.x, (pos + 1u) & qm, pin);
    }
    // New blocks enter the small queue, or the main queue where the ghost
    // remembers them, deepest first.
    PC_RUNS_FN void insert_s3(uint32_t r, uint32_t np, vu pid, vu pl, vu pc, uint32_t hend, uint32_t nw, uint32_t m) {
        const vu zu = wv.vu0(0);
        const vb isn = (pl > 0u) & (pc + pl > hend);
        const vu off = W::sel(isn & (wv.vu0(hend) > pc), wv.vu0(hend) - pc, zu);
        const vu a = pid + off, L = W::sel(isn, pl - off, zu);
        uint32_t ng = 0;
        if (P.g_cap > 0) ng = match<true, false, true>(gh, 0, 0, np, a, L, zu);
        if (general) return;
        const uint64_t nmask = W::ballot(isn);
        const uint32_t nnew = (uint32_t)W::popc(nmask);
        if (!room_for<true>(q0, nnew + ng)) return;
        uint32_t nghost = 0;
        if (ng == 0) {
            const vu at = (wv.vu0(q0.tail + nnew - 1u) - W::mbcnt(nmask)) & qm;
            W::st(isn, q0.lo, at, a);
            W::st(isn, q0.w, at, L | nw);
            W::st(isn, q0.x, at, wv.vu0(r));
            q0.tail += nnew;
        } else {
            if (!room_for<true>(q1, ng)) return;
            W::sync();
            const vb inl = lane < ng;
            const vu glo = W::ld(xlo, lane & 63u), gl = W::ld(xw, lane & 63u) & kLen, gi = W::ld(xi, lane & 63u);
            for (uint64_t pm = nmask; pm; ) {
                const int i = 63 - W::clz(pm);
                pm &= ~(1ull << i);
                const uint32_t lo = W::rdl(a, i);
                uint32_t end = lo + W::rdl(L, i);
                uint64_t gm = W::ballot(inl & (gi == (uint32_t)i));
                while (gm) {       // the ghost's parts of this piece, deepest first
                    const vu key = W::sel(W::of_mask(gm), glo - lo + 1u, zu);
                    const uint32_t top = W::wmax(key);
                    const int l = W::ffs(W::ballot(key == top) & gm);
                    gm &= ~(1ull << l);
                    const uint32_t x0 = W::rdl(glo, l), xl = W::rdl(gl, l);
                    if (x0 + xl < end) push(q0, x0 + xl, (end - x0 - xl) | nw, r, true);
                    push(q1, x0, xl | nw, r, true);
                    nghost += xl;
                    end = x0;
                }
                if (end > lo) push(q0, lo, (end - lo) | nw, r, true);
            }
        }
        s_size += (int32_t)(m - nghost);
        s_unp += (int32_t)(m - nghost);
        m_unp += (int32_t)nghost;
        s3_ghits += nghost;
    }
};

}  // namespace pcr
