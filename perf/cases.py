"""Timed cases of the hot path: block cutting and chained keys
(device.cut_and_hash) and batched cache replay (device.ReplayBatch), over the
sizes, trace shapes, policies and options that users of the package run.

Two kinds of case:

  hash     cut_and_hash of one device-resident set of requests.
  replay   ReplayBatch.launch of `traces` traces x their instances; with
           "step" the keys are computed in the pass too, as in bench.py.

Trace shapes (`shape`) follow the recipes of tracegen.py (same length laws,
hot sets, group and prefix structure), drawn here with numpy for the
structure and torch on the GPU for the token ids, so that full-size inputs
are made in well under a second:

  onetouch   victim with 32 hot prefixes against a polluter of unique prompts
  twopass    the polluter's prompts come back once
  delayed    8 groups: 6 benign with private prefixes, victim, polluter phases
  tiny       4 hot 512-token prefixes against unique 512-token prompts
  attack     4 hot 1,536-token prefixes, polluter with unique or twice-sent prompts
  selector   unique prompts of about 31 blocks from many groups
  chat       multi-turn conversations, every turn re-sending its context (views
             into the conversation's own tokens)
  tiers      several groups on three service contracts, with arrival ticks
  chunks     the engine's own keys, not chained: requests are lists of document
             chunks whose blocks have the same keys at any position

Everything the path computes is an integer, so all outputs compare exactly.
"""
import numpy as np
import torch

from paper_2608_01657_amd import PC_STATS_RECORD_BYTES
from paper_2608_01657_amd import device as dv
from paper_2608_01657_amd import tracegen as tg

DEV = "cuda"
LRU, S3, PS, SQ = tg.POLICY_LRU, tg.POLICY_S3FIFO, tg.POLICY_PREFIXSHIELD, tg.POLICY_STATICQUOTA


# --------------------------------------------------------------------------
# Cases
# --------------------------------------------------------------------------

def listed():
    return [
        # keys of the requests that arrived in one scheduler tick of a serving engine
        dict(name="hash_tick", kind="hash", shape="mixed", requests=48, mean_tokens=700, traces=1),
        # a few long documents (retrieval, code): long serial chains, few requests
        dict(name="hash_long", kind="hash", shape="mixed", requests=96, mean_tokens=60000, traces=1),
        # a trace archive of unique prompts, streamed from HBM once
        dict(name="hash_onetouch", kind="hash", shape="onetouch", requests=50000, traces=8),
        # conversations: aliased views, every turn re-reads its context
        dict(name="hash_chat", kind="hash", shape="chat", requests=50000, traces=16),
        # smallest named workload: one small cache, three policies (debugging, unit studies)
        dict(name="replay_tiny", kind="replay", shape="tiny", requests=4000, traces=1, capacity=256, mix="three"),
        # the policy comparison on the one-touch traces, per seed, keys included
        dict(name="step_onetouch", kind="replay", shape="onetouch", requests=20000, traces=16, capacity=4096,
             mix="three", step=True),
        # the benchmark's batch: 1,024 concurrent instances, a refill-rate sweep, keys included
        dict(name="step_scale1024", kind="replay", shape="onetouch", requests=50000, traces=16, capacity=4096,
             mix="sweep62", step=True),
        # capacity planning on conversations: five cache sizes x three policies
        dict(name="replay_chat", kind="replay", shape="chat", requests=20000, traces=64, capacity=0, mix="capacities"),
        # the debt-gate ablation: 8 groups, 8 refill rates, long trace
        dict(name="replay_delayed", kind="replay", shape="delayed", requests=40000, traces=8, capacity=4096,
             mix="rates8"),
        # the attack table: every policy and ablation at the paper's cache size, with
        # per-request outcomes for the confidence intervals
        dict(name="replay_attack", kind="replay", shape="attack", requests=4000, traces=10, capacity=511,
             mix="ablations", per_request=True),
        # tenants on three contracts, bursty arrival ticks, per-request outcomes
        dict(name="replay_tiers", kind="replay", shape="tiers", requests=20000, traces=8, capacity=4096,
             mix="tiers", per_request=True),
        # keys from another engine that are not chained (the same chunk at any position)
        dict(name="replay_chunks", kind="replay", shape="chunks", requests=8000, traces=4, capacity=3000,
             mix="three"),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    if rng.random() < 0.3:
        shape = rng.choice(["mixed", "mixed", "onetouch", "chat", "twopass"])
        if shape == "mixed":
            mean = _log(rng, 20, 60000)
            return dict(kind="hash", shape=shape, requests=_log(rng, 1, min(100000, max(2, 40_000_000 // mean))),
                        mean_tokens=mean, traces=1)
        return dict(kind="hash", shape=shape, requests=_log(rng, 500, 40000), traces=rng.randint(1, 8))
    shape = rng.choice(["onetouch", "twopass", "delayed", "tiny", "attack", "selector", "chat", "tiers", "chunks"])
    case = dict(kind="replay", shape=shape, requests=_log(rng, 100, 20000), traces=rng.randint(1, 8),
                capacity=_log(rng, 96, 20000))
    case["mix"] = {"onetouch": "sweep13", "delayed": "rates8", "attack": "ablations", "tiers": "tiers"}.get(
        shape, rng.choice(["three", "ablations"]))
    if shape == "selector":
        case["groups"] = rng.choice([3, 8, 32, 64])
    if rng.random() < 0.3:
        case["per_request"] = True
    if shape != "chunks" and rng.random() < 0.3:
        case["step"] = True
    return case


# --------------------------------------------------------------------------
# Trace structure (host) and tokens (device)
# --------------------------------------------------------------------------

class _Trace:
    """Request descriptors of one trace.  A request's tokens are either hot
    prefix `hot` (an index, or -1) followed by fresh tokens at `off` of its
    trace's stream, or a view of tokens that are already there."""

    def __init__(self, n_groups):
        self.n_groups = n_groups
        self.contract = None
        self.tick = None
        self.hot = None          # [R] hot prefix of the request, -1: none
        self.hot_len = np.zeros(0, np.int64)
        self.n_tokens = 0


def _zipf(rng, s, n, size):
    w = np.arange(1, n + 1, dtype=np.float64) ** (-s)
    return rng.choice(n, size=size, p=w / w.sum())


def _lognormal(rng, mu, sigma, size, lo, hi):
    return np.clip(np.floor(np.exp(rng.normal(mu, sigma, size))), lo, hi).astype(np.int64)


def _laid_out(t, lens, hot, hot_len, group, prefix, view=None):
    """Stream layout: every request has its own tokens, except those with
    view[r] >= 0, which alias request view[r]."""
    own = np.ones(len(lens), bool) if view is None else view < 0
    off = np.concatenate([[0], np.cumsum(np.where(own, lens, 0))])
    t.n_tokens = int(off[-1])
    off = off[:-1].copy()
    if view is not None:
        off[~own] = off[view[~own]]
        hot = np.where(own, hot, -1)      # an alias copies nothing
    t.off, t.length, t.hot, t.hot_len = off, lens, hot, np.asarray(hot_len, np.int64)
    t.group, t.prefix, t.n_prefix = group, prefix, int(prefix.max()) + 1 if len(prefix) else 1
    return t


def _attack_like(rng, own, role, hot_len, s, suffix, pol_len, view_of=None):
    """Victim requests (role 0: a hot prefix + suffix fresh tokens) against a
    polluter (role 1: unique prompts; view_of(k): the earlier polluter prompt
    that polluter request k sends again, or -1)."""
    n = len(role)
    pol = np.flatnonzero(role == 1)
    z = np.zeros(n, np.int64)
    z[role == 0] = own.permutation(_zipf(rng, s, len(hot_len), n - len(pol)))
    lens = np.where(role == 0, hot_len[z] + suffix, 0)
    view = np.full(n, -1, np.int64)
    pid = np.arange(len(pol))
    if view_of is not None:
        src = np.array([view_of(k) for k in range(len(pol))], np.int64)
        again = src >= 0
        view[pol[again]] = pol[src[again]]
        pid[again] = src[again]
    lens[pol] = pol_len(len(pol)) if view_of else own.permutation(pol_len(len(pol)))
    lens[view >= 0] = lens[view[view >= 0]]
    prefix = np.where(role == 0, z, 0)
    prefix[pol] = len(hot_len) + pid
    return _laid_out(_Trace(2), lens, np.where(role == 0, z, -1), hot_len, role, prefix, view)


def _structure(case, seed, i):
    """Trace i of the case.  Its lengths are drawn for the case, and what has
    which of them (the order of hot prefixes, prompts and groups) from the
    seed, so that every seed gives as many keys."""
    n, shape = case["requests"], case["shape"]
    rng, own = np.random.default_rng([n, case["traces"], i]), np.random.default_rng([seed, i])
    r = np.arange(n)
    polluter = lambda k: _lognormal(rng, 7.6, 0.5, k, 256, 8192)
    if shape == "mixed":
        lens = np.maximum(1, rng.exponential(case["mean_tokens"], n)).astype(np.int64)
        if n > 2:
            lens[rng.integers(0, n)] = 15      # a request without a full block
        return _laid_out(_Trace(8), own.permutation(lens), np.full(n, -1), [], own.integers(0, 8, n), r)
    if shape == "onetouch":
        return _attack_like(rng, own, (r % 4 != 0).astype(np.int64), rng.integers(1024, 4097, 32), 0.9, 128, polluter)
    if shape == "twopass":
        uniq = (n // 2 + 1) // 2
        return _attack_like(rng, own, r % 2, rng.integers(1024, 4097, 32), 0.9, 128, polluter,
                            lambda k: k - uniq if k >= uniq else -1)
    if shape == "tiny":
        return _attack_like(rng, own, r % 2, np.full(4, 512), 1.0, 64, lambda k: np.full(k, 512))
    if shape == "attack":
        role = ((r % 2 == 1) & (r >= n // 10)).astype(np.int64)
        twice = (lambda k: k - 1 if k % 2 else -1) if i % 2 else None
        return _attack_like(rng, own, role, np.full(4, 1536), 1.0, 64, lambda k: np.full(k, 1536), twice)
    if shape == "selector":
        G = case.get("groups", 8)
        w = np.arange(1, G + 1, dtype=np.float64)
        return _laid_out(_Trace(G), own.permutation(_lognormal(rng, 6.2, 0.5, n, 128, 2048)), np.full(n, -1), [],
                         own.choice(G, size=n, p=w / w.sum()), r)
    if shape == "delayed":
        f = r / n
        pol = ((f < 0.2) | ((f >= 0.45) & (f < 0.65))) & (r % 4 == 3)
        group = np.where(pol, 7, rng.integers(0, 7, n))
        hot_len = np.concatenate([np.full(48, 2048), rng.integers(1024, 4097, 32)])
        hot = np.where(group < 6, 8 * group + _zipf(rng, 1.1, 8, n), 48 + _zipf(rng, 0.9, 32, n))
        mix = own.permutation(np.flatnonzero(~pol))
        group[~pol], hot[~pol] = group[mix], hot[mix]
        hot = np.where(pol, -1, hot)
        lens = np.where(pol, 0, hot_len[np.maximum(hot, 0)] + 128)
        p = np.flatnonzero(pol)
        uniq = max(1, int((p < 0.2 * n).sum()))
        lens[p] = polluter(len(p))
        view = np.full(n, -1, np.int64)
        k = np.arange(len(p))
        again = k >= uniq
        view[p[again]] = p[(k[again] - uniq) % uniq]
        lens[view >= 0] = lens[view[view >= 0]]
        prefix = np.where(pol, 0, hot)
        prefix[p] = 80 + np.where(again, (k - uniq) % uniq, k)
        t = _laid_out(_Trace(8), lens, hot, hot_len, group, prefix, view)
        return t
    if shape == "tiers":
        group = rng.choice(6, size=n, p=[0.20, 0.15, 0.15, 0.15, 0.15, 0.20])
        hot_len = np.concatenate([rng.integers(1024, 4097, 32), np.full(24, 2048)])
        z8, z32 = _zipf(rng, 1.1, 8, n), _zipf(rng, 0.9, 32, n)
        mix = own.permutation(n)
        group, z8, z32 = group[mix], z8[mix], z32[mix]
        hot = np.where(group == 0, z32, np.where(group < 4, 32 + 8 * (group - 1) + z8, -1))
        lens = np.where(hot >= 0, hot_len[np.maximum(hot, 0)] + 128, 0)
        fresh = np.flatnonzero(hot < 0)
        lens[fresh] = own.permutation(polluter(len(fresh)))
        prefix = np.where(hot >= 0, hot, 0)
        prefix[fresh] = 56 + np.arange(len(fresh))
        t = _laid_out(_Trace(6), lens, hot, hot_len, group, prefix)
        t.contract = np.choose(group, [0, 1, 2, np.where(z8 < 4, 1, 2), 0, 2])
        t.tick = np.cumsum(own.integers(0, 3, n)) // 8 * 8
        return t
    if shape == "chat":
        G, active = 16, 4
        group, slot = rng.integers(0, G, n), rng.integers(0, active, n)
        stream = group * active + slot
        order = np.argsort(stream, kind="stable")         # requests of one slot, in time order
        first = np.concatenate([[0], np.flatnonzero(np.diff(stream[order])) + 1, [n]])
        starts = []                                       # where a new conversation begins (in `order`)
        for a, b in zip(first[:-1], first[1:]):
            at = a + np.concatenate([[0], np.cumsum(rng.integers(2, 11, b - a))])
            starts.append(at[at < b])
        starts = np.concatenate(starts)
        conv = np.cumsum(np.isin(np.arange(n), starts)) - 1
        user, reply = _lognormal(rng, 4.5, 1.0, n, 1, 1 << 14), _lognormal(rng, 5.5, 0.8, n, 1, 1 << 14)
        run = np.cumsum(user + reply)
        ctx = run - (run - user - reply)[starts][conv] - reply      # context up to this user turn
        lens = np.minimum(ctx, 16384)
        size = np.zeros(len(starts), np.int64)
        np.maximum.at(size, conv, lens)
        base = np.concatenate([[0], np.cumsum(size)])
        t = _Trace(G)
        t.off, t.length, t.prefix = np.empty(n, np.int64), np.empty(n, np.int64), np.empty(n, np.int64)
        t.off[order], t.length[order], t.prefix[order] = base[conv], lens, conv
        t.group, t.n_prefix, t.n_tokens = own.permutation(G)[group], len(starts), int(base[-1])
        t.hot = np.full(n, -1)
        return t
    raise ValueError(shape)


def _fill(tokens, t, gen):
    """Token ids of one trace: uniform, with each hot prefix copied in front
    of the requests that carry it."""
    tokens.random_(0, tg.VOCAB, generator=gen)
    req = np.flatnonzero(t.hot >= 0)
    if not len(req):
        return
    hot = torch.randint(0, tg.VOCAB, (int(t.hot_len.sum()),), generator=gen, device=DEV, dtype=torch.int32)
    base = np.concatenate([[0], np.cumsum(t.hot_len)])[:-1]
    L = torch.from_numpy(t.hot_len[t.hot[req]]).to(DEV)
    end = torch.cumsum(L, 0)
    which = torch.repeat_interleave(torch.arange(len(req), device=DEV), L)
    at = torch.arange(int(end[-1]), device=DEV) - (end - L)[which]
    dst, src = torch.from_numpy(t.off[req]).to(DEV)[which] + at, torch.from_numpy(base[t.hot[req]]).to(DEV)[which] + at
    tokens[dst] = hot[src]


def _chunk_traces(case, seed):
    """Unchained keys: documents of 4..31 blocks, Zipf-popular, 1..8 of them a
    request in any order (the same one now and then twice), then a unique
    question of 1..8 blocks."""
    out = []
    for i in range(case["traces"]):
        rng = np.random.default_rng([seed, i, 77])
        n, docs, G = case["requests"], 2000, 8
        size = rng.integers(4, 32, docs)
        base = np.concatenate([[0], np.cumsum(size)])
        k = rng.integers(1, 9, n)
        pick = _zipf(rng, 0.8, docs, int(k.sum()))
        q = rng.integers(1, 9, n)
        # parts in request order: its documents, then its question
        part_req = np.concatenate([np.repeat(np.arange(n), k), np.arange(n)])
        start = np.concatenate([base[pick], base[-1] + np.concatenate([[0], np.cumsum(q)])[:-1]])
        length = np.concatenate([size[pick], q])
        order = np.argsort(part_req, kind="stable")
        start, length, part_req = start[order], length[order], part_req[order]
        ident = np.repeat(start - np.concatenate([[0], np.cumsum(length)])[:-1], length) + np.arange(length.sum())
        mixed = rng.integers(1, 1 << 63, dtype=np.int64) | 1
        keys = (ident.astype(np.uint64) + 1) * np.uint64(mixed)
        keys ^= keys >> np.uint64(29)
        off = np.concatenate([[0], np.cumsum(np.bincount(part_req, weights=length, minlength=n).astype(np.int64))])
        group = rng.integers(0, G, n)
        out.append(tg.KeyTrace(keys, off, group.astype(np.uint8), np.zeros(n, np.uint8),
                               (group * 4 + rng.integers(0, 4, n)).astype(np.uint32), G, 4 * G))
    return out


def _device_traces(case, seed):
    """One DeviceTrace over all traces of the case, and each trace's rows."""
    ts = [_structure(case, seed, i) for i in range(case["traces"])]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    tok_base = np.concatenate([[0], np.cumsum([t.n_tokens for t in ts])])
    tokens = torch.empty(int(tok_base[-1]), dtype=torch.int32, device=DEV)
    for t, a, b in zip(ts, tok_base[:-1], tok_base[1:]):
        _fill(tokens[a:b], t, gen)
    cat = lambda xs, dt: torch.from_numpy(np.ascontiguousarray(np.concatenate(xs).astype(dt))).to(DEV)
    zero = lambda t: np.zeros(len(t.off), np.int64)
    d = dv.DeviceTrace(
        tokens=tokens, tok_off=cat([t.off + a for t, a in zip(ts, tok_base)], np.int64),
        length=cat([t.length for t in ts], np.int32), ns=cat([t.group for t in ts], np.int32),
        group=cat([t.group for t in ts], np.uint8),
        contract=cat([zero(t) if t.contract is None else t.contract for t in ts], np.uint8),
        prefix=cat([t.prefix for t in ts], np.int32),
        tick=None if ts[0].tick is None else cat([t.tick for t in ts], np.int64),
        n_groups=max(t.n_groups for t in ts), n_prefix=max(t.n_prefix for t in ts),
        max_req_blocks=max(int(t.length.max()) // 16 for t in ts))
    return d, ts


def _instances(case, seed=0):
    """Replay instances of one trace (trace index 0); the seed moves the
    refill rates a little (below 2 % of a block per tick)."""
    out = _named_instances(case)
    for x in out:
        x.contracts = [(rho + seed * 7919 % 1021, beta) for rho, beta in x.contracts]
    return out


def _named_instances(case):
    C, mix = case["capacity"], case["mix"]
    three = (LRU, S3, PS)
    beta = tg.DEFAULT_BETA_Q16
    if mix == "three":
        return [tg.Instance(0, p, C) for p in three]
    if mix == "capacities":
        return [tg.Instance(0, p, c) for c in (1024, 2048, 4096, 8192, 16384) for p in three]
    if mix.startswith("sweep"):
        return [tg.Instance(0, LRU, C), tg.Instance(0, S3, C)] + [
            tg.Instance(0, PS, C, contracts=[(k * tg.Q16 // 4, beta)]) for k in range(1, int(mix[5:]) + 1)]
    if mix == "rates8":
        return [tg.Instance(0, p, C, contracts=[((1 << k) * tg.Q16, beta)])
                for k in range(8) for p in three]
    if mix == "ablations":
        return [tg.Instance(0, p, C) for p in three] + [
            tg.Instance(0, PS, C, flags=tg.FLAG_NO_SEGMENTATION), tg.Instance(0, PS, C, flags=tg.FLAG_NO_DEBT_GATE),
            tg.Instance(0, SQ, C)]
    if mix == "tiers":
        c = list(tg.TIER_CONTRACTS)
        return [tg.Instance(0, p, C, contracts=c) for p in three] + [
            tg.Instance(0, S3, C, contracts=c, s3_small_permille=250, s3_move_threshold=2),
            tg.Instance(0, PS, C, contracts=c, eps_q16=4 * tg.Q16)]
    raise ValueError(mix)


def prepare(case, seed):
    if case["shape"] == "chunks":
        d, views = None, [dv.upload_keys(kt, DEV) for kt in _chunk_traces(case, seed)]
    else:
        d, ts = _device_traces(case, seed)
        dv.cut_and_hash(d)                    # sizes the key buffer
        if case["kind"] == "hash":
            return dict(trace=d, batch=None, step=True)
        base = np.concatenate([[0], np.cumsum([len(t.off) for t in ts])])
        views = [dv.TraceView(keys=d.keys[:d.n_keys], key_off=d.key_off[a:b + 1], group=d.group[a:b],
                              contract=d.contract[a:b], prefix=d.prefix[a:b],
                              tick=None if d.tick is None else d.tick[a:b], n_groups=t.n_groups,
                              n_prefix=t.n_prefix, max_req_blocks=int(t.length.max()) // 16, n_keys=d.n_keys)
                 for t, a, b in zip(ts, base[:-1], base[1:])]
    insts = []
    for i in range(len(views)):
        for x in _instances(case, seed):
            x.trace = i
            insts.append(x)
    batch = dv.ReplayBatch(views, insts, per_request=case.get("per_request", False))
    return dict(trace=d, batch=batch, step=case.get("step", False))


def run(state):
    d, batch = state["trace"], state["batch"]
    out = []
    if state["step"]:
        dv.cut_and_hash(d, n_keys=d.n_keys)
        out += [d.key_off, d.keys[:d.n_keys], d.status]
    if batch is not None:
        batch.launch()
        out.append(batch.stats)
        if batch.per_request is not None:
            out.append(batch.per_request)
    return out


# --------------------------------------------------------------------------
# What a pass cannot do without, and how close its outputs have to be
# --------------------------------------------------------------------------

_MEAN_TOKENS = dict(onetouch=2330, twopass=2490, delayed=2270, tiny=544, attack=1570, selector=560, chat=1620,
                    tiers=2340)


def work(case):
    """Token and key traffic of one pass from the shapes' mean lengths: hash
    reads each token once and writes each key, replay reads each key and
    request descriptor once (however many instances share them) and writes
    the stats records and per-request outcomes."""
    n = case["requests"] * case["traces"]
    mean = case.get("mean_tokens") or _MEAN_TOKENS.get(case["shape"], 1000)
    if case["shape"] == "chunks":
        mean = 16 * 83
    keys = n * mean / 16
    once = {"chat": 0.25, "twopass": 0.75}.get(case["shape"], 1.0)     # share of the tokens not re-sent
    total = 0.0
    if case["kind"] == "hash" or case.get("step"):
        total += n * mean * 4 * once + keys * 8 + n * 32
    if case["kind"] == "replay":
        inst = len(_instances(case)) * case["traces"]
        total += keys * 8 + n * 14 + inst * PC_STATS_RECORD_BYTES
        if case.get("per_request"):
            total += 16 * case["requests"] * inst
    return {"bytes": total, "flops": 0.0}


def tolerance(case):
    return "exact"
