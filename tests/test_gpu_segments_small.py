"""The segment builder of up to 4096 rows over up to 256 keys: both sides of its row and key limits, tiles of 16 and 32
rows, one key, all keys, one hot key, rows without adapter and ids outside the pool."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
from harness import to_dev
from test_gpu_segments import compare

pytestmark = pytest.mark.gpu

BAD_ADAPTER, BAD_EXPERT = 1, 2           # bits of the status word


def build(rank, n, E, aid, eid):
    P = aid.size
    desc = L.PoolDesc(n, 1, E, [(8, 8)], rank)
    slab = torch.empty(L.lora_pool_bytes(desc), dtype=torch.uint8, device="cuda")
    pool = L.lora_register_pool(desc, slab)
    seg = L.Segments(P)
    for t in (seg.perm, seg.seg_start, seg.seg_key, seg.tiles, seg.counts):
        t.fill_(-7)
    seg.status.fill_(5)
    L.lora_build_segments(pool, to_dev(aid), None if eid is None else to_dev(eid), P, seg)
    torch.cuda.synchronize()
    return seg


@pytest.mark.parametrize("P", [1, 63, 65, 1023, 1024, 1025, 2048, 2049, 4095, 4096, 4097])
@pytest.mark.parametrize("n,E", [(1, 1), (2, 1), (85, 3), (32, 8), (257, 1)])
@pytest.mark.parametrize("kind", ["even", "hot", "few", "bad"])
def test_small_builder(P, n, E, kind):
    r = np.random.default_rng(P * 7 + n)
    aid, eid = r.integers(0, n, P).astype(np.int32), r.integers(0, E, P).astype(np.int32)
    if kind == "hot":                        # one key has nine rows of ten, one row of 13 has no adapter
        hot = r.random(P) < 0.9
        aid[hot], eid[hot] = n - 1, E - 1
        aid[::13] = -1
    elif kind == "few":                      # the first and the last key only
        aid, eid = np.where(aid % 2, n - 1, 0).astype(np.int32), np.where(aid % 2, E - 1, 0).astype(np.int32)
    elif kind == "bad":
        aid[::5], eid[3::7] = n + 3, -2
    seg = build(16, n, E, aid, eid if E > 1 else None)
    want_status = 0
    if kind == "bad":
        bad_a, bad_e = aid >= n, (eid < 0) & (E > 1)
        want_status = BAD_ADAPTER * int(bad_a.any()) | BAD_EXPERT * int(bad_e.any())
        aid, eid = np.where(bad_a | bad_e, -1, aid).astype(np.int32), np.where(bad_e, 0, eid).astype(np.int32)
    compare(seg, aid, eid if E > 1 else None, n, E)
    assert int(seg.status.cpu()[0]) == want_status


@pytest.mark.parametrize("P,n", [(4096, 8), (2048, 64), (3001, 5)])
def test_small_builder_with_tiles_of_32_rows(P, n):
    aid = np.sort(np.random.default_rng(P).integers(0, n, P)).astype(np.int32)
    seg = build(64, n, 1, aid, None)
    assert seg.c.tile_rows == 32
    compare(seg, aid, None, n, 1)
