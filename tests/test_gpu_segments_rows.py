"""The counting path's rows per thread: batch sizes around every form and around the pairs of rows that its larger forms leave
out, batches that it hands to the radix path together with their keys, and what a row more than a form takes may cost."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
from harness import to_dev
from test_gpu_segments import compare, make_pool, run_segments

pytestmark = pytest.mark.gpu

EDGES = [1, 63, 1024, 1025, 2047, 2049, 4095, 6143, 6144, 6145, 8191, 10239, 10241, 12287, 12289, 14335, 14337, 16383]


@pytest.mark.parametrize("P", EDGES)
@pytest.mark.parametrize("n,E", [(300, 1), (9000, 1), (200, 128)])
def test_edges_of_the_forms(P, n, E):
    rng = np.random.default_rng(P)
    aid = rng.integers(-1, n, size=P).astype(np.int32)
    aid[0], aid[-1] = n - 1, 0
    eid = rng.integers(0, E, size=P).astype(np.int32) if E > 1 else None
    compare(run_segments(make_pool(n, E), aid, eid), aid, eid, n, E)


@pytest.mark.parametrize("P", [257, 1500, 4000, 7000, 9000, 11000])
@pytest.mark.parametrize("n", [3000, 65536])
def test_handed_to_the_radix_path(P, n):
    """One key of 256 rows or more, beside rows without adapter and with ids outside the pool (reported, and left out)."""
    rng = np.random.default_rng(P + n)
    aid = rng.integers(-1, n, size=P).astype(np.int32)
    aid[rng.permutation(P)[:max(256, P // 5)]] = n - 1
    bad = np.nonzero(aid != n - 1)[0][:1]
    aid[bad] = n + 7
    seg = run_segments(make_pool(n, 1), aid, None)
    compare(seg, np.where(aid < n, aid, -1).astype(np.int32), None, n, 1)
    assert int(seg.status.cpu()[0]) == (1 if bad.size else 0)


def test_a_row_more_than_a_form_takes():
    """8192 and 8193 rows over 4096 keys: 1.11 of the time; 1.31 with a form that does the work of 16384 rows."""
    pool, us = make_pool(4096, 1), {}
    for P in (8192, 8193):
        ids, seg, times = to_dev(np.random.default_rng(1).integers(0, 4096, P).astype(np.int32)), L.Segments(P), []
        stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.stream(stream):
            L.lora_build_segments(pool, ids, None, P, seg)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(40):
                L.lora_build_segments(pool, ids, None, P, seg)
        for _ in range(15):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            graph.replay()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 1e3 / 40)
        us[P] = sorted(times)[7]
    print("us by rows:", us)
    assert us[8193] <= 1.21 * us[8192], us
