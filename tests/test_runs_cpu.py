"""The run-based replay (csrc/pc_runs.h) on the CPU, its wavefront run lane
by lane with every LDS access bounds-checked (runs_host.cpp), against the
oracle: every counter and every request's outcome, over the trace shapes of
the package, crafted keys with duplicates, orphans and unchained repeats, and
rings small enough that an instance must be handed to the general kernel."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
from gpu_util import POLICIES, many_groups_batch, random_key_batch, step_boundary_batch
from paper_2608_01657_amd import GROUP_FIELDS, INST_FIELDS
from paper_2608_01657_amd import tracegen as tg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
P, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("runs") / "librunshost.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-Wno-unknown-pragmas", "-shared", "-fPIC",
                    "-I", os.path.join(ROOT, "paper_2608_01657_amd", "csrc"),
                    os.path.join(ROOT, "tests", "runs_host.cpp"), "-o", so], check=True)
    L = ctypes.CDLL(so)
    L.runs_host_replay.restype = ctypes.c_int
    L.runs_host_replay.argtypes = [P, P, P, P, P, P, i64, i32, i64, i32, i64, i32, i32, P, P, i64, i32, i32, i32,
                                   i64, P, i64, i32, i32, P, P, P]
    u32, f32 = ctypes.c_uint32, ctypes.c_float
    L.runs_host_pays.argtypes = [i32, i32, i32, i64, u32, u32, u32, u32, f32, f32]
    L.runs_host_batch_pays.argtypes = [u32, f32, f32, f32, f32]
    L.runs_host_sample.argtypes = [P, i64, P]
    L.runs_host_is_sampled.argtypes = [i64, i64]
    return L


def _ptr(a):
    return None if a is None else a.ctypes.data_as(P)


def run_host(L, kt, inst, window=0, other=None, ahead=0, interleave=0):
    """(groups, inst, per_request), or when it is left to the general kernel, by
    whom ("analysis", before any request is replayed, or "replay").
    other: key offsets of a second trace on the same key buffer, analysed
    behind this one or ahead of it."""
    a = [np.ascontiguousarray(x, t) for x, t in ((kt.keys if kt.keys.size else np.zeros(1), np.uint64),
                                                 (kt.key_off, np.int64), (kt.group, np.uint8),
                                                 (kt.contract, np.uint8), (kt.prefix, np.uint32))]
    tick = None if kt.tick is None else np.ascontiguousarray(kt.tick, np.int64)
    rho = np.array([c[0] for c in inst.contracts], np.int64)
    beta = np.array([c[1] for c in inst.contracts], np.int64)
    R = kt.n_req
    off2 = None if other is None else np.ascontiguousarray(other, np.int64)
    gs = np.zeros((kt.n_groups, len(GROUP_FIELDS)), np.int64)
    st = np.zeros(len(INST_FIELDS), np.int64)
    pr = np.zeros((R, 4), np.int32)
    rc = L.runs_host_replay(*map(_ptr, a), _ptr(tick), R, kt.n_groups, kt.n_prefix, inst.policy, inst.capacity,
                            inst.flags, len(inst.contracts), _ptr(rho), _ptr(beta), inst.eps_q16,
                            inst.s3_small_permille, inst.s3_move_threshold, window, kt.keys.size, _ptr(off2),
                            0 if other is None else len(other) - 1, ahead, interleave, _ptr(gs), _ptr(st), _ptr(pr))
    if rc:
        return {1: "replay", 2: "analysis"}[rc]
    return [dict(zip(GROUP_FIELDS, map(int, row))) for row in gs], dict(zip(INST_FIELDS, map(int, st))), pr


def compare(L, kt, inst, window=0, label="", **shared):
    """1 if the instance finished, equal to the oracle's; 0 if it was left."""
    got = run_host(L, kt, inst, window, **shared)
    if isinstance(got, str):
        return 0
    o = oracle.replay_key_trace(kt, inst, per_request=True)
    what = f"{label} {tg.POLICY_NAMES[inst.policy]} C={inst.capacity} flags={inst.flags}"
    bad = np.flatnonzero((got[2] != o.per_request).any(axis=1))
    assert bad.size == 0, f"{what}: request {bad[0]}: {got[2][bad[0]]} != {o.per_request[bad[0]]}"
    for g, (a, b) in enumerate(zip(got[0], o.groups)):
        assert a == b, f"{what} group {g}: {a} != {b}"
    assert got[1] == o.inst, what
    return 1


def key_trace(tr):
    keys, off = oracle.hash_trace(tr)
    return tg.KeyTrace(keys, off, tr.group, tr.contract, tr.prefix, tr.n_groups, tr.n_prefix, tr.tick)


def batch(L, kts, per, window=0):
    done = total = 0
    for i, (kt, insts) in enumerate(zip(kts, per)):
        for inst in insts:
            done += compare(L, kt, inst, window, f"trace {i}")
            total += 1
    return done, total


@pytest.mark.parametrize("chunk", range(4))
def test_random_keys(host, chunk):
    done, total = batch(host, *random_key_batch(chunk))
    assert done > 0.6 * total      # (a request of more than 64 pieces is left to the general kernel)


def test_many_groups(host):
    done, total = batch(host, *many_groups_batch())
    assert done == total


def test_long_requests_of_random_keys_are_left_or_exact(host):
    batch(host, *step_boundary_batch())


@pytest.mark.parametrize("name,seeds,n,caps", [
    ("tiny", [0], 1500, (256, 64, 31)), ("onetouch4096", [0, 1], 1200, (4096, 700, 200)),
    ("twopass", [0], 1000, (4096, 500)), ("delayed", [0], 3000, (4096, 1000)), ("tiers", [0], 1500, (4096, 800)),
    ("chat", [0], 3000, (1024, 4096, 300)), ("chat_bursty", [0], 2000, (2048, 150)),
    ("attack_replay", [0], 1500, (511, 97)), ("selector512x8", [0], 1500, (512, 40)),
    ("selector4096x32", [0], 1500, (4096, 600))])
def test_workloads(host, name, seeds, n, caps):
    traces, insts = tg.workload(name, seeds=seeds, n_requests=n)
    for ti, tr in enumerate(traces):
        kt = key_trace(tr)
        for inst in insts:
            if inst.trace != ti:
                continue
            for cap in caps:
                x = tg.Instance(0, inst.policy, cap, contracts=inst.contracts, flags=inst.flags,
                                eps_q16=inst.eps_q16)
                assert compare(host, kt, x, 0, name) == 1
        for cap in caps:
            for x in (tg.Instance(0, tg.POLICY_STATICQUOTA, cap, contracts=insts[0].contracts),
                      tg.Instance(0, tg.POLICY_S3FIFO, cap, contracts=insts[0].contracts, s3_small_permille=400,
                                  s3_move_threshold=2)):
                assert compare(host, kt, x, 0, name) == 1


def chunk_trace(seed, n_req=500, docs=60, doc_len=(1, 12), n_groups=4):
    """Unchained keys: a request is a list of documents (with repeats, and
    now and then only a document's start), then a question of its own."""
    rng = np.random.default_rng(seed)
    size = rng.integers(*doc_len, docs)
    base = 1000 * np.arange(1, docs + 1)
    keys, off = [], [0]
    for r in range(n_req):
        for d in rng.integers(0, docs, rng.integers(0, 7)) ** 2 // docs:
            k = int(size[d]) if rng.random() < 0.8 else int(rng.integers(1, size[d] + 1))
            keys.extend(base[d] + np.arange(k))
        keys.extend(10_000_000 + 100 * r + np.arange(rng.integers(0, 5)))
        off.append(len(keys))
    group = rng.integers(0, n_groups, n_req)
    return tg.KeyTrace(np.array(keys, np.uint64) * np.uint64(0x9E3779B97F4A7C15), np.array(off, np.int64),
                       group.astype(np.uint8), np.zeros(n_req, np.uint8),
                       (group * 3 + rng.integers(0, 3, n_req)).astype(np.uint32), n_groups, 3 * n_groups)


@pytest.mark.parametrize("seed", range(6))
def test_unchained_documents(host, seed):
    kt = chunk_trace(seed)
    for pol in POLICIES:
        for cap in (20, 90, 300, 2000):
            for flags in ([0, 1, 2, 3] if pol == tg.POLICY_PREFIXSHIELD else [0]):
                assert compare(host, kt, tg.Instance(0, pol, cap, flags=flags, contracts=[(tg.Q16 * 3, 20 * tg.Q16)]),
                               0, f"chunks {seed}") == 1


@pytest.mark.parametrize("window", [256, 512])
def test_small_windows_are_exact_or_left(host, window):
    """LDS windows far below the planner's: they compact often, and an
    instance either overflows (left) or is exact."""
    left = n = 0
    for seed in range(4):
        kt = chunk_trace(100 + seed, n_req=400, docs=200)
        for pol in POLICIES:
            for cap in (40, 150, 400, 1200):
                left += 1 - compare(host, kt, tg.Instance(0, pol, cap), window, f"window {window}")
                n += 1
    assert 0 < left < n if window == 256 else left < n // 2


def test_single_block_pieces(host):
    """40 pieces of one block a request, in an order of its own."""
    rng = np.random.default_rng(5)
    reqs = [rng.permutation(300)[:40] for _ in range(200)]
    kt = tg.KeyTrace(np.concatenate(reqs).astype(np.uint64), 40 * np.arange(201, dtype=np.int64),
                     rng.integers(0, 3, 200).astype(np.uint8), np.zeros(200, np.uint8), np.zeros(200, np.uint32), 3, 1)
    for pol in POLICIES:
        for cap in (50, 70, 150, 290):
            assert compare(host, kt, tg.Instance(0, pol, cap), 0, "pieces") == 1


def test_widest_windows(host):
    """Single-block prompts, a run each: more than the first windows hold,
    exact in the widest ones."""
    reqs = [[10 * r] if r % 3 else [10 * r, 7, 8] for r in range(3500)]
    n = len(reqs)
    kt = tg.KeyTrace(np.array([k for r in reqs for k in r], np.uint64),
                     np.cumsum([0] + [len(r) for r in reqs]).astype(np.int64), (np.arange(n) % 3).astype(np.uint8),
                     np.zeros(n, np.uint8), (np.arange(n) % 50).astype(np.uint32), 3, 50)
    for pol in POLICIES:
        assert compare(host, kt, tg.Instance(0, pol, 6000 if pol == tg.POLICY_STATICQUOTA else 2500)) == 0
        assert compare(host, kt, tg.Instance(0, pol, 2500), -1) == 1


def partial_repeats(seed, n_req=120, docs=60):
    """Requests that hold a document's beginning and, more than 64 blocks of
    their own later, the whole document (or the other way round).  Few of
    them share a document, so that a cut that one misses is missed."""
    rng = np.random.default_rng(seed)
    reqs = []
    for r in range(n_req):
        d = 1000 * (1 + r % docs)
        parts = [np.arange(d, d + int(rng.integers(1, 11))), np.arange(d, d + 10)]
        own = 100_000 + 500 * r + np.arange(int(rng.integers(60, 140)))
        a, b = parts if rng.random() < 0.7 else parts[::-1]
        reqs.append(np.concatenate([a, own, b]))
    group = rng.integers(0, 3, n_req)
    return tg.KeyTrace(np.concatenate(reqs).astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15),
                       np.cumsum([0] + [len(x) for x in reqs]).astype(np.int64), group.astype(np.uint8),
                       np.zeros(n_req, np.uint8), group.astype(np.uint32), 3, 3)


@pytest.mark.parametrize("interleave", [0, 1, 2, 3])
def test_partial_repeats_while_other_requests_add_cuts(host, interleave):
    """Cuts that other wavefronts add between two steps of a request's listing
    change nothing in it."""
    kt = partial_repeats(interleave)
    for pol in POLICIES:
        for cap in (60, 700):
            assert compare(host, kt, tg.Instance(0, pol, cap), 0, "repeats", interleave=interleave) == 1


def _on_keys(keys, off):
    n = len(off) - 1
    g = np.arange(n) % 3
    return tg.KeyTrace(keys, np.asarray(off, np.int64), g.astype(np.uint8), np.zeros(n, np.uint8),
                       g.astype(np.uint32), 3, 3)


def ends_inside():
    """Two traces of 20 requests on one key buffer, the same ten keys again and
    again; the last request of the second one ends half way."""
    keys = np.tile(np.arange(1, 11), 20).astype(np.uint64)
    off = 10 * np.arange(21)
    return _on_keys(keys, off), _on_keys(keys, np.concatenate([off[:-1], [195]]))


def random_cuts(seed):
    """Two traces on one key buffer of repeated documents, cut at random (some
    starts in common); the last request of the second starts where one of the
    first does."""
    rng = np.random.default_rng(seed)
    keys = np.concatenate([1000 * d + np.arange(1, 25) for d in rng.integers(0, 9, 90)]).astype(np.uint64)
    off, other = (np.unique(np.concatenate([[0], 12 * rng.integers(0, 178, n)])) for n in (50, 40))
    k = int(rng.choice(np.flatnonzero(np.isin(other, off))[1:]))
    return _on_keys(keys, off), _on_keys(keys, np.concatenate([other[:k + 1], [other[k] + rng.integers(1, 30)]]))


@pytest.mark.parametrize("ahead", [0, 1])
def test_equal_starts_with_different_ends(host, ahead):
    """Requests of two traces that start at one position and end at different
    ones keep their pieces in the same place: whichever is listed last, an
    instance of either is exact."""
    done = n = 0
    for pair in [ends_inside()] + [random_cuts(s) for s in range(12)]:
        for kt, other in (pair, pair[::-1]):
            for pol in POLICIES:
                for cap in (7, 64, 300):
                    done += compare(host, kt, tg.Instance(0, pol, cap), 0, "shared", other=other.key_off, ahead=ahead)
                    n += 1
    assert done >= n // 2


@pytest.mark.parametrize("pieces", [64, 65])
def test_too_many_pieces_are_left_by_the_analysis(host, pieces):
    """One request that takes single blocks of many earlier ones, at the end of
    the trace: 64 pieces finish on runs, 65 are left before the first request."""
    reqs = [np.arange(100 * r, 100 * r + 9) for r in range(pieces)]
    reqs.append(np.array([100 * r for r in range(pieces)]))
    n = len(reqs)
    kt = tg.KeyTrace(np.concatenate(reqs).astype(np.uint64), np.cumsum([0] + [len(x) for x in reqs]).astype(np.int64),
                     (np.arange(n) % 3).astype(np.uint8), np.zeros(n, np.uint8), np.zeros(n, np.uint32), 3, 1)
    for pol in POLICIES:
        if pieces == 64:
            assert compare(host, kt, tg.Instance(0, pol, 200)) == 1
        else:
            assert run_host(host, kt, tg.Instance(0, pol, 200)) == "analysis"


def test_contracts_out_of_range_are_left_by_the_analysis(host):
    kt = chunk_trace(3, n_req=50)
    kt.contract[49] = 2
    one = (tg.Q16, 20 * tg.Q16)
    for pol in POLICIES:
        assert compare(host, kt, tg.Instance(0, pol, 90, contracts=[one] * 3)) == 1
        assert run_host(host, kt, tg.Instance(0, pol, 90, contracts=[one] * 2)) == "analysis"


# us a request, one instance alone on an MI355X: (policy, C, blocks of a
# document, documents of a request, on runs, in the general kernels); 1,500
# requests of documents out of 3 C / d
MEASURED = [
    (0, 256, 4, 16, 5.4, 5.9), (0, 1024, 1, 60, 33.5, 5.9), (0, 1024, 8, 24, 7.6, 6.0), (0, 4096, 1, 24, 35.3, 5.1),
    (0, 4096, 1, 60, 89.0, 5.2), (0, 4096, 4, 24, 15.0, 5.1), (0, 4096, 16, 4, 2.5, 4.9), (0, 4096, 32, 16, 5.4, 10.2),
    (0, 4096, 32, 60, 16.3, 35.0), (0, 16384, 1, 60, 265.0, 7.0), (0, 16384, 4, 24, 36.5, 7.2),
    (1, 256, 16, 4, 4.9, 11.1), (1, 1024, 1, 60, 70.1, 11.2), (1, 1024, 32, 16, 13.9, 23.8),
    (1, 4096, 2, 60, 100.6, 10.4), (1, 4096, 4, 24, 30.5, 9.9), (1, 4096, 32, 60, 44.4, 78.4),
    (1, 16384, 8, 60, 101.2, 31.2), (2, 256, 16, 16, 6.4, 12.6), (2, 1024, 1, 60, 35.5, 10.4),
    (2, 4096, 1, 60, 96.0, 9.0), (2, 4096, 8, 8, 6.3, 8.6), (2, 4096, 32, 60, 26.2, 72.0), (2, 16384, 2, 60, 174.6, 17.9),
    (3, 4096, 1, 60, 86.9, 6.2), (3, 4096, 16, 4, 2.3, 5.5), (3, 4096, 32, 16, 4.9, 14.1)]


@pytest.mark.parametrize("policy,cap,d,k,runs,general", MEASURED)
def test_form_of_many_pieces(host, policy, cap, d, k, runs, general):
    """The rule takes the faster form where one is much faster, also where the
    chip is shared (in the general kernels `load` times, with the widest
    windows `rounds` times)."""
    n, distinct = 1500, 3 * cap // d
    fresh = int(distinct * (1 - (1 - 1 / distinct) ** (n * k)))
    for load, rounds in ((1, 1), (2.2, 4)):
        pays = host.runs_host_pays(policy, cap, 4, n, n, n * k, n * k * d, fresh, load, rounds)
        for bit, r, g in ((1, 1, load), (2, 1, 1), (4, rounds, load)):
            if runs * r > 1.7 * general * g:
                assert not pays & bit
            if runs * r < 0.6 * general * g:
                assert pays & bit


def test_form_of_a_batch(host):
    """Both forms one after the other, or all instances in one of them."""
    f = host.runs_host_batch_pays
    # (longest on runs of those that pay, in the general kernels of the rest; of all)
    for pays in (0, 1, 7):
        assert f(pays, 4, 7, 30, 12) == pays
        assert f(pays, 4, 7, 11.5, 12) == pays
        assert f(pays, 4, 7, 11.5, 7.5) == 0
        assert f(pays, 0.5, 7, 20, 7) == pays        # (not worth less than a tenth)
        assert f(pays, 5, 5, 6, 7) == 7
        assert f(pays, 5, 0, 5, 20) == pays
        assert f(pays, 0, 9, 40, 9) == pays


def test_sampled_requests(host):
    """One of every 64th part, or all; as many of every kind of request that
    comes in a fixed rhythm."""
    for n in (1, 16, 63, 64, 65, 127, 128, 129, 1000, 5000, 50_000, 65_536):
        r = np.flatnonzero([host.runs_host_is_sampled(r, n) for r in range(n)])
        assert len(r) == n if n <= 64 else 32 <= len(r) <= 64
        if n >= 1000:
            assert np.bincount(r % 4, minlength=4).min() >= 9 and np.bincount(r % 2, minlength=2).min() >= 22


def test_sums_of_a_sample(host):
    """The largest values of 64 requests fit their fields."""
    sums = np.zeros(4, np.uint32)
    rng = np.random.default_rng(1)
    for req in (np.tile([64, 64, 1 << 20], (64, 1)), np.tile([0, 0, 0], (64, 1)), np.zeros((0, 3), int),
                np.stack([rng.integers(0, 65, 64), rng.integers(0, 65, 64), rng.integers(0, 70_000, 64)], 1)):
        req = np.ascontiguousarray(req, np.int64)
        host.runs_host_sample(_ptr(req), len(req), _ptr(sums))
        assert list(sums) == [len(req), req[:, 0].sum(), req[:, 1].sum(), np.minimum(req[:, 2], 65535).sum()]
