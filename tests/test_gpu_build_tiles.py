"""Tile records of segments of many lengths where the batch is sorted inside the first shrink: up to three tiles of a
key are written by the thread that owns it, the rest by its wave."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
from harness import to_dev
from test_gpu_segments import compare

pytestmark = pytest.mark.gpu

LENGTHS = [[1792, 47, 48, 49, 64, 48], [2048], [1, 1047, 1000], [49] * 41, [33, 0, 48, 0, 49, 0, 1000, 16, 17]]


@pytest.mark.parametrize("lengths", LENGTHS)
@pytest.mark.parametrize("first_key", [0, 61, 200])
def test_long_segments_inside_the_shrink(lengths, first_key):
    n = 256
    aid = np.repeat(first_key + np.arange(len(lengths)), lengths).astype(np.int32)
    aid = np.random.default_rng(len(lengths)).permutation(aid) if len(lengths) != 6 else aid
    P = aid.size
    desc = L.PoolDesc(n, 1, 1, [(136, 136)], 16)
    slab = torch.zeros(L.lora_pool_bytes(desc), dtype=torch.uint8, device="cuda")
    pool = L.lora_register_pool(desc, slab)
    assert L.lora_build_apply_launches(pool, 0, 1, P) <= 2
    seg = L.Segments(P)
    for t in (seg.perm, seg.seg_start, seg.seg_key, seg.tiles):
        t.fill_(-7)
    x = torch.zeros(P, 136, dtype=torch.bfloat16, device="cuda")
    y = torch.ones(P, 136, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(L.lora_group_ws_bytes(pool, 0, 1, P), dtype=torch.uint8, device="cuda")
    L.lora_build_apply_group(pool, 0, 0, x, 136, None, to_dev(aid), None, P, seg, [y], [136], ws)
    torch.cuda.synchronize()
    compare(seg, aid, None, n, 1)
    assert bool((y == 1).all())
