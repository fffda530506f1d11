"""The replay on runs and its trace analysis on the GPU, where they can go
wrong: key buffers that several traces share or overlap in, duplicates that
add cuts, instances that must be handed to the general kernel (too many runs,
too many pieces, a malformed request), a workspace too small for the
analysis, and the edges of a wavefront (63-65 pieces and requests)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_01657_amd as P
from gpu_util import POLICIES, _pad_trace, assert_same, run_key_traces
from paper_2608_01657_amd import device as dv
from paper_2608_01657_amd import tracegen as tg
from test_runs_cpu import chunk_trace, ends_inside, partial_repeats, random_cuts

pytestmark = pytest.mark.gpu
GENERAL, RUNS, WIDE = P.PC_ROUTE_GENERAL, P.PC_ROUTE_RUNS, P.PC_ROUTE_RUNS_WIDE


def _insts(caps, pols=POLICIES, contracts=((tg.Q16 * 2, 30 * tg.Q16),)):
    return [tg.Instance(0, p, c, contracts=list(contracts)) for p in pols for c in caps]


def _trace(reqs, n_groups=3, seed=0):
    rng = np.random.default_rng(seed)
    n = len(reqs)
    g = rng.integers(0, n_groups, n)
    return tg.KeyTrace(np.concatenate([np.asarray(r, np.uint64) for r in reqs] + [np.zeros(0, np.uint64)]),
                       np.cumsum([0] + [len(r) for r in reqs]).astype(np.int64), g.astype(np.uint8),
                       np.zeros(n, np.uint8), (g * 2 + rng.integers(0, 2, n)).astype(np.uint32), n_groups,
                       2 * n_groups)


@pytest.mark.parametrize("seed", range(3))
def test_unchained_documents_and_duplicates(seed):
    run_key_traces([chunk_trace(seed, n_req=700)], [_insts((25, 300, 3000))], routes=[RUNS] * 12)


@pytest.mark.parametrize("seed", range(3))
def test_partial_repeats_far_apart_in_a_request(seed):
    """Every request adds cuts to documents that other wavefronts are listing."""
    run_key_traces([partial_repeats(seed, n_req=3000, docs=1500)], [_insts((60, 700, 4096))], routes=[RUNS] * 12)


@pytest.mark.parametrize("n_req", [1, 15, 16, 17, 63, 64, 65])
def test_shortest_traces_on_runs(n_req):
    run_key_traces([chunk_trace(50 + n_req, n_req=n_req)], [_insts((1, 7, 64, 4096))],
                   routes=[RUNS if n_req >= 16 else GENERAL] * 16)


@pytest.mark.parametrize("blocks", [63, 64, 65, 130])
def test_requests_of_single_block_pieces(blocks):
    """Every block its own piece (no two requests repeat an order): the general
    kernel replays them several times faster."""
    rng = np.random.default_rng(blocks)
    reqs = [rng.permutation(400)[:blocks] for _ in range(90)]
    run_key_traces([_trace(reqs)], [_insts((64, 150, 500))], routes=[GENERAL] * 12)


@pytest.mark.parametrize("pieces", [63, 64, 65])
def test_a_request_of_single_block_pieces(pieces):
    """The last of many short requests has a piece for each lane, or more."""
    reqs = [np.arange(10 * r, 10 * r + 7) for r in range(300)] + [10 * np.arange(pieces) * 4 + 3]
    run_key_traces([_trace(reqs)], [_insts((64, 150, 500, 3000))], routes=[RUNS if pieces <= 64 else GENERAL] * 16)


def _documents(d, k, docs, n):
    """n requests of k documents of d blocks."""
    rng = np.random.default_rng([d, k, docs])
    return _trace([np.concatenate([100 * x + np.arange(d) for x in rng.integers(0, docs, k)]) for _ in range(n)])


@pytest.mark.parametrize("d,k,docs,caps,route", [(30, 3, 400, (300, 4096), RUNS), (4, 8, 2000, (300,), RUNS),
                                                 (1, 40, 6000, (300, 4096), GENERAL), (2, 12, 12000, (16384,), GENERAL)])
def test_form_follows_the_pieces(d, k, docs, caps, route):
    """Long documents, and many short ones (at 16,384 blocks a piece is compared
    with more runs)."""
    run_key_traces([_documents(d, k, docs, 800)], [_insts(caps)], routes=[route] * 4 * len(caps))


def test_form_of_a_batch_of_both():
    """The general kernels begin when the replay on runs has ended: a batch takes
    both forms, or the general kernels for all where that is over earlier."""
    long, short = _documents(30, 3, 400, 3000), _documents(1, 40, 6000, 200)
    run_key_traces([long, short], [_insts((300, 4096)), _insts((300, 4096))], routes=[RUNS] * 8 + [GENERAL] * 8)
    near = _documents(4, 8, 2000, 800)
    run_key_traces([near, _documents(1, 40, 6000, 800)], [_insts((300,)), _insts((300,))], routes=[GENERAL] * 8)


def test_more_runs_than_rings_hold():
    """Single-block prompts: thousands of runs are live at once, and more in
    the ghost of S3-FIFO than any window holds."""
    reqs = [[10 * r] if r % 3 else [10 * r, 7, 8] for r in range(6000)]
    run_key_traces([_trace(reqs)], [_insts((500, 4096, 9000))],
                   routes=[RUNS, WIDE, WIDE] + [RUNS, GENERAL, GENERAL] + 2 * [RUNS, WIDE, WIDE])


@pytest.mark.parametrize("cap", [257, 310, 383, 384, 769, 840, 1793, 1860])
def test_general_kernels_log_beside_a_full_cache(cap):
    """Capacities a little above a power of two, short requests: 256 entries of
    the free-queue log have to stay free beside a full cache, which S3-FIFO
    scans past (the general kernels replay the batch too)."""
    kt = chunk_trace(cap, n_req=700, docs=60 if cap < 700 else 250)
    run_key_traces([kt], [[tg.Instance(0, tg.POLICY_S3FIFO, cap, s3_small_permille=p, s3_move_threshold=t)
                           for p, t in ((100, 1), (100, 0), (250, 2), (1000, 1))] + _insts((cap,))])


def test_malformed_request_after_many_good_ones():
    kt = chunk_trace(9, n_req=200)
    ok, bad = chunk_trace(10, n_req=150), chunk_trace(11, n_req=150)
    bad.group[120] = 200
    dts = [dv.upload_keys(k) for k in (kt, ok, bad)]
    insts = [tg.Instance(t, p, 100) for t in range(3) for p in POLICIES]
    b = dv.ReplayBatch(dts, insts)
    b.launch()
    assert b.routes() == [RUNS] * 8 + [GENERAL] * 4
    for (groups, inst, status), x in zip(b.results(), insts):
        if x.trace == 2:
            assert status == P.PC_EINVAL and not any(inst.values())
        else:
            assert_same((groups, inst, status), oracle.replay_key_trace((kt, ok)[x.trace], x))


def _views(kt, dt, ranges):
    """Traces of request ranges of one uploaded key trace, on its key buffer."""
    out, kts = [], []
    for a, b in ranges:
        out.append(dv.TraceView(keys=dt.keys[:dt.n_keys], key_off=dt.key_off[a:b + 1], group=dt.group[a:b],
                                contract=dt.contract[a:b], prefix=dt.prefix[a:b], tick=None, n_groups=kt.n_groups,
                                n_prefix=kt.n_prefix, max_req_blocks=dt.max_req_blocks, n_keys=dt.n_keys))
        kts.append(tg.KeyTrace(kt.keys, kt.key_off[a:b + 1], kt.group[a:b], kt.contract[a:b], kt.prefix[a:b],
                               kt.n_groups, kt.n_prefix))
    return out, kts


def test_traces_that_share_and_overlap_in_one_key_buffer():
    kt = chunk_trace(21, n_req=600)
    dt = dv.upload_keys(kt)
    views, kts = _views(kt, dt, [(0, 600), (0, 300), (300, 600), (150, 450), (599, 600)])
    # the same keys cut into requests elsewhere: starts inside other requests
    off = np.unique(np.concatenate([[0], np.sort(np.random.default_rng(3).integers(0, kt.keys.size, 400)),
                                    [kt.keys.size]])).astype(np.int64)
    n = len(off) - 1
    other = tg.KeyTrace(kt.keys, off, np.zeros(n, np.uint8), np.zeros(n, np.uint8), np.zeros(n, np.uint32),
                        kt.n_groups, kt.n_prefix)
    o = dv.upload_keys(other)
    o.keys = dt.keys
    # (the trace of a request that starts inside another's pieces is left)
    for batch, ks, runs in ((views, kts, range(5)), (views + [o], kts + [other], [4])):
        insts = [tg.Instance(t, p, c) for t in range(len(batch)) for p in POLICIES for c in (60, 700)]
        b = dv.ReplayBatch(batch, insts, per_request=True)
        b.launch()
        assert b.routes() == [RUNS if x.trace in runs else GENERAL for x in insts]
        pr = b.per_request_arrays()
        for k, (res, x) in enumerate(zip(b.results(), insts)):
            w = oracle.replay_key_trace(ks[x.trace], x, per_request=True)
            assert_same(res, w, f"instance {k}")
            assert np.array_equal(pr[k], w.per_request)


def test_small_views_of_a_large_key_buffer():
    """Traces that can read a part of their key buffer only are analysed over
    that part: at its start, inside, overlapping, at its end; malformed
    offsets leave their trace alone."""
    kt = chunk_trace(22, n_req=3000)
    dt = dv.upload_keys(kt)
    views, kts = _views(kt, dt, [(0, 40), (100, 140), (130, 150), (2000, 2100), (2984, 3000)])
    assert sum(k.n_req * dt.max_req_blocks for k in kts) < dt.n_keys
    for k, wrong in ((0, -5), (16, dt.n_keys + 9), (3, 0), (0, dt.n_keys + 40)):
        bad, badk = _views(kt, dt, [(500, 516)])
        off = badk[0].key_off.copy()
        off[k] = wrong
        bad[0].key_off = torch.from_numpy(off).to(dt.key_off.device)
        views += bad
        kts.append(None)
    insts = [tg.Instance(t, p, c) for t in range(len(views)) for p in POLICIES for c in (60, 700)]
    b = dv.ReplayBatch(views, insts, per_request=True)
    b.launch()
    assert b.routes() == [RUNS if kts[x.trace] else GENERAL for x in insts]
    pr = b.per_request_arrays()
    for k, (res, x) in enumerate(zip(b.results(), insts)):
        if kts[x.trace] is None:
            assert res[2] == P.PC_EINVAL
            continue
        w = oracle.replay_key_trace(kts[x.trace], x, per_request=True)
        assert_same(res, w, f"instance {k}")
        assert np.array_equal(pr[k], w.per_request)


@pytest.mark.parametrize("order", [(0, 1), (1, 0)])
def test_equal_starts_with_different_ends(order):
    """The last request of a trace ends inside another trace's request that
    starts where it does; and random cuts of one key buffer."""
    # (with random cuts requests of one trace start inside the other's pieces)
    for kts, runs in (ends_inside(), (0, 1)), (random_cuts(0), (1,)), (random_cuts(1), (0,)):
        dts = [dv.upload_keys(k) for k in kts]
        for d in dts:
            d.keys = dts[0].keys
        kts, dts = [kts[i] for i in order], [dts[i] for i in order]
        insts = [tg.Instance(t, p, c) for t in range(2) for p in POLICIES for c in (7, 64, 300)]
        # (beside instances of an empty trace, since a batch this small would
        # take the general kernels for both traces)
        dts.append(dv.upload_keys(_pad_trace()))
        full = insts + [tg.Instance(2, tg.POLICY_PREFIXSHIELD, 4096) for _ in range(2000)]
        b = dv.ReplayBatch(dts, full, per_request=True)
        b.launch()
        assert b.routes()[:len(insts)] == [RUNS if order[x.trace] in runs else GENERAL for x in insts]
        pr = b.per_request_arrays()
        for k, (res, x) in enumerate(zip(b.results(), insts)):
            w = oracle.replay_key_trace(kts[x.trace], x, per_request=True)
            assert_same(res, w, f"instance {k}")
            assert np.array_equal(pr[k], w.per_request)


def test_general_kernel_where_the_workspace_has_no_room_for_the_analysis():
    """A workspace of the general kernels' size is accepted, and so is the
    static entry for a batch whose analysis does not fit its array."""
    tr = tg.onetouch_4096(2000, 1500)
    t = dv.upload(tr)
    dv.cut_and_hash(t)
    insts = [tg.Instance(0, p, c) for p in POLICIES for c in (256, 4096)]
    b = dv.ReplayBatch([t], insts)
    need = P.pc_replay_workspace_bytes(b.tdesc, b.idesc)
    # the run plan adds at least the table and the ids of every key
    small = b.workspace[:(need - 12 * t.n_keys) // 8 // 32 * 32]
    stats = torch.zeros_like(b.stats)
    assert P.pc_replay_route_offset(b.tdesc, b.idesc, small.numel() * 8) == 0
    P.pc_replay_batch(b.tdesc, b.idesc, small, stats)
    b.launch()
    assert b.routes() == [RUNS] * 8
    torch.cuda.synchronize()
    assert torch.equal(stats, b.stats)
    big = tg.onetouch_4096(2001, 50000)
    T = dv.upload(big)
    dv.cut_and_hash(T)
    B = dv.ReplayBatch([T], insts[:2])
    assert P.pc_replay_workspace_bytes(B.tdesc, B.idesc) > P.PC_STATIC_WORKSPACE_BYTES
    B.launch()
    assert B.routes() == [RUNS] * 2
    stats = torch.zeros_like(B.stats)
    P.pc_replay_batch_static(B.tdesc, B.idesc, stats)
    torch.cuda.synchronize()
    assert torch.equal(stats, B.stats)
