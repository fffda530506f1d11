"""Keys and offsets of calls with few or long requests on the GPU, where a
workgroup takes a request: lengths around its steps (64 blocks a wavefront,
64 x 4, 8 or 16 a workgroup), each rule of the dispatch and its edges, and
the one-launch offsets up to and past their last size.  Whole numbers:
every key and offset equals the oracle's."""
import numpy as np
import pytest

from paper_2608_01657_amd import tracegen as tg
from test_gpu_parity import _check_hash

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 63, 64, 65, 127, 128, 255, 256, 257, 511, 512, 513, 575, 1023, 1024, 1025, 2047, 2048, 2049, 2111]


def _trace(n_req, avg, shared, seed):
    """n_req requests of avg blocks in the mean, edges among them; `shared`:
    all are views of one short token range."""
    rng = np.random.default_rng(seed)
    e = np.array([b for b in EDGES if b <= 3 * avg])
    nb = rng.integers(0, 2 * avg + 1, n_req)
    pick = rng.random(n_req) < 0.3
    nb[pick] = rng.choice(e, int(pick.sum()))
    nb[-1] = max(0, n_req * avg - int(nb[:-1].sum()))       # the mean is avg where the others allow it
    lens = (nb * 16 + rng.integers(0, 16, n_req)).astype(np.int32)
    if shared:
        n_tok = int(lens.max()) + 1024
        offs = rng.integers(0, n_tok - lens + 1)
    else:
        offs = np.cumsum(np.concatenate([[rng.integers(0, 4)], lens[:-1]]))
        n_tok = int(offs[-1] + lens[-1])
    toks = rng.integers(-2**31, 2**31, n_tok, dtype=np.int64).astype(np.int32)
    return tg.Trace("teams", toks, offs.astype(np.int64), lens, rng.integers(0, 256, n_req).astype(np.uint8),
                    np.zeros(n_req, np.uint8), np.zeros(n_req, np.uint32), 256, n_req)


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("n_req,avg", [(1, 1), (1, 65), (3, 383), (1, 384), (40, 700), (7, 1535), (1, 1536), (12, 2500),
                                       (512, 100), (513, 100), (513, 520), (600, 511), (700, 767), (520, 800),
                                       (4096, 540), (4097, 540)])
def test_hash_team_edges(n_req, avg, shared):
    _check_hash(_trace(n_req, avg, shared, 31 * n_req + avg))


@pytest.mark.parametrize("n_req", [2, 1023, 4096, 4097, 8191, 8192, 8193, 32767, 32768])
def test_offsets_sizes(n_req):
    _check_hash(_trace(n_req, 2, False, n_req))
