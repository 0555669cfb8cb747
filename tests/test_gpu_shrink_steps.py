"""Ends of the decode shrink's K range: inputs shorter than a step, ranges that end inside one, columns beyond the
row's end inside a K-block, and rows with infinities and NaN, which must stay in their own rows."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
import workloads as W
from gpu_common import oracle_projection
from harness import DeviceBatch, DevicePool, bits_from_dev, to_dev

pytestmark = pytest.mark.gpu

HEIGHTS = [1, 3, 5, 16, 17]


@pytest.mark.parametrize("rank", [8, 16, 32, 64])
@pytest.mark.parametrize("h_in", [8, 40, 136, 520, 1032, 2600])
@pytest.mark.parametrize("streamed", [False, True])
def test_ends_of_the_range(rank, h_in, streamed):
    n, tokens = len(HEIGHTS), sum(HEIGHTS)
    w = W.Workload("t", "dense", n, 1, 1, rank, tuple(W.Proj(f"p{i}", h_in, 136, "x") for i in range(2)), tokens, "zipf", 1.0)
    b = W.make_batch(w, 9, y_mode="normal", hetero_scale=True)
    b.adapter_id[:] = np.random.default_rng(9).permutation(np.repeat(np.arange(n), HEIGHTS))
    ws = W.make_weights(w, 9, bank_elems=1 << 20)
    bad = [int(np.nonzero(b.adapter_id == a)[0][0]) for a in (1, 3, 4)]      # one row of three of the tiles
    x = b.inputs["x"]
    x[bad[0], 0], x[bad[1], h_in - 1], x[bad[2], h_in // 2] = 0x7FC0, 0x7F80, 0xFF80      # NaN, inf, -inf
    dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
    L.lora_pool_set_activation_policy(dp.pool, L.LORA_ACT_STREAMING if streamed else L.LORA_ACT_RESIDENT)
    ok = np.ones(tokens, bool)
    ok[bad] = False
    with np.errstate(invalid="ignore"):
        want = [oracle_projection(b, ws, 0, j, use_y=False).delta for j in range(2)]
    # two projections in one launch, then one
    L.lora_build_segments(dp.pool, to_dev(b.adapter_id), None, tokens, db.seg)
    xd = db.inputs["x"]
    for group in ((0, 1), (0,)):
        size = L.lora_group_ws_bytes(dp.pool, 0, len(group), tokens)
        y = [torch.zeros(tokens, 136, dtype=torch.float32, device="cuda") for _ in group]
        L.lora_apply_group(dp.pool, 0, 0, xd, h_in, None, db.seg, y, [136] * len(group),
                           torch.empty(size, dtype=torch.uint8, device="cuda"), L.LORA_DTYPE_F32)
        for j in group:
            got = y[j].cpu().numpy().astype(np.float64)
            assert not np.isfinite(got[~ok]).any()
            # fp32 sums over K and the two-part bf16 operand: 1e-5 of the whole
            assert np.linalg.norm(got[ok] - want[j][ok]) <= 1e-5 * np.linalg.norm(want[j][ok])
