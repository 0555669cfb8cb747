"""The segment builder's counting path at the edges of its forms: rows per thread, counter words per thread, four 8-bit
counters in a word (255 rows of a key are counted, 256 are handed to the radix path) and several workgroups, bit for bit."""
import numpy as np
import pytest

from test_gpu_segments import compare, make_pool, run_segments

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1, 1023, 1025, 2048, 4096, 4097, 8192, 8193, 16384])
@pytest.mark.parametrize("n,E", [(257, 1), (4096, 1), (4097, 1), (64, 128), (8193, 1), (128, 128), (16385, 1), (256, 128), (32769, 1)])
def test_rows_and_keys(P, n, E):
    rng = np.random.default_rng(P + n)
    p = np.arange(1, n + 1, dtype=np.float64) ** -0.7
    aid = rng.choice(n, size=P, p=p / p.sum()).astype(np.int32)
    aid[rng.random(P) < 0.05] = -1
    aid[-1] = n - 1
    eid = rng.integers(0, E, size=P).astype(np.int32) if E > 1 else None
    compare(run_segments(make_pool(n, E), aid, eid), aid, eid, n, E)


@pytest.mark.parametrize("counts", [[255, 255, 255, 255], [254, 256, 1, 0], [255, 0, 256, 0], [1, 1, 1, 256], [0, 255, 0, 257],
                                    [16, 17, 15, 33], [512, 512, 0, 0]])
@pytest.mark.parametrize("more", [0, 1500, 6000])
def test_full_counters(counts, more):
    """Keys 400 .. 403 share a word; beside them rows of other keys, for one and for several workgroups."""
    rng = np.random.default_rng(sum(counts) + more)
    n = 3000
    aid = np.concatenate([np.repeat(np.arange(400, 404), counts), rng.integers(0, 396, 1), rng.integers(404, n, more)])
    aid = rng.permutation(aid).astype(np.int32)
    compare(run_segments(make_pool(n, 1), aid, None), aid, None, n, 1)
