"""Which work items the long-segment shrink takes, at the edges of the rule: one projection around 48 and 96 rows per key with up to
64 keys and more, and two projections over a key space beyond the segment list of the kernel of blocks, of which few occur: blocks
of one segment in the other kernel."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
import workloads as W
from gpu_common import oracle_projection
from harness import DeviceBatch, DevicePool
from test_gpu_long_blocks import run_lengths

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [16, 32, 64])
@pytest.mark.parametrize("lengths", [[1024] * 5, [1 + i % 3 for i in range(4000)] + [513, 130, 33]])
def test_few_segments_of_a_large_key_space(lengths, rank, monkeypatch):
    monkeypatch.setenv("LORA_TILE_ROWS", "32")
    dp, db = run_lengths(lengths, rank, (136, 40), 392, 5, "normal", True, n=5000)
    assert min(5000, db.P) > 4096 and int(db.seg.counts[0].cpu()) <= 4096


@pytest.mark.parametrize("rank", [32, 64])
@pytest.mark.parametrize("keys,mean", [(64, 47), (64, 48), (65, 48), (64, 95), (65, 95), (65, 96)])
def test_rows_per_key(keys, mean, rank, monkeypatch):
    monkeypatch.setenv("LORA_TILE_ROWS", "32")
    lengths = np.random.default_rng(mean).multinomial(keys * mean, np.arange(1, keys + 1) ** -0.5 / (np.arange(1, keys + 1) ** -0.5).sum())
    n, P, h_in = keys, keys * mean, 200
    w = W.Workload("t", "dense", n, 1, 1, rank, (W.Proj("p", h_in, 8, "x"),), P, "uniform")
    b = W.make_batch(w, 6, y_mode="zero")
    b.adapter_id[:] = np.random.default_rng(1).permutation(np.repeat(np.arange(n, dtype=np.int32), lengths))
    ws = W.make_weights(w, 6, bank_elems=1 << 20)
    dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
    L.lora_build_segments(dp.pool, db.adapter_id, None, P, db.seg)
    assert db.seg.c.tile_rows == 32
    x, y = db.inputs["x"], torch.zeros(P, 8, dtype=torch.float32, device="cuda")
    v = torch.full((L.lora_v_bytes(dp.pool, 0, P),), 0xFF, dtype=torch.uint8, device="cuda")
    L.lora_shrink(dp.pool, 0, 0, x, h_in, None, db.seg, v)
    L.lora_expand(dp.pool, 0, 0, v, db.seg, y, 8, L.LORA_DTYPE_F32)
    want = oracle_projection(b, ws, 0, 0, use_y=False).delta
    # fp32 sums over K and the two-part bf16 operand: 1e-5 of the whole
    assert np.linalg.norm(y.cpu().numpy().astype(np.float64) - want) <= 1e-5 * np.linalg.norm(want)
