"""The long-segment shrink over blocks of one segment, whose x and A go straight into LDS a stage (64 K values) or two
ahead: K ranges of one, two, three and more stages, ranges that end inside one and inside a K-block, with anything
behind the end of a row, and rows with infinities and NaN, which must stay in their own rows."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
import workloads as W
from gpu_common import oracle_projection
from harness import DeviceBatch, DevicePool, to_dev

pytestmark = pytest.mark.gpu

LENGTHS = [200, 129, 64, 33]                  # 106 rows per key: blocks also for one projection


@pytest.mark.parametrize("rank", [16, 32, 64])
@pytest.mark.parametrize("h_in", [8, 40, 64, 72, 128, 136, 200, 1000])
def test_ends_of_the_range(rank, h_in, monkeypatch):
    monkeypatch.setenv("LORA_TILE_ROWS", "32")
    n, tokens = len(LENGTHS), sum(LENGTHS)
    w = W.Workload("t", "dense", n, 1, 1, rank, tuple(W.Proj(f"p{i}", h_in, 136, "x") for i in range(2)), tokens, "zipf", 1.0)
    b = W.make_batch(w, 9, y_mode="normal", hetero_scale=True)
    b.adapter_id[:] = np.random.default_rng(9).permutation(np.repeat(np.arange(n), LENGTHS))
    ws = W.make_weights(w, 9, bank_elems=1 << 20)
    bad = [int(np.nonzero(b.adapter_id == a)[0][-1]) for a in (0, 2, 3)]
    x = b.inputs["x"]
    x[bad[0], 0], x[bad[1], h_in - 1], x[bad[2], h_in // 2] = 0x7FC0, 0x7F80, 0xFF80      # NaN, inf, -inf
    dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
    ok = np.ones(tokens, bool)
    ok[bad] = False
    with np.errstate(invalid="ignore"):
        want = [oracle_projection(b, ws, 0, j, use_y=False).delta for j in range(2)]
    L.lora_build_segments(dp.pool, to_dev(b.adapter_id), None, tokens, db.seg)
    assert db.seg.c.tile_rows == 32
    xd = torch.full((tokens, h_in + 64), 0x7FC0, dtype=db.inputs["x"].dtype, device="cuda")      # bits: NaN behind the rows
    xd[:, :h_in] = db.inputs["x"]
    for group in ((0, 1), (0,)):
        ws_buf = torch.full((L.lora_group_ws_bytes(dp.pool, 0, len(group), tokens),), 0xFF, dtype=torch.uint8, device="cuda")
        y = [torch.zeros(tokens, 136, dtype=torch.float32, device="cuda") for _ in group]
        L.lora_apply_group(dp.pool, 0, 0, xd, xd.shape[1], None, db.seg, y, [136] * len(group), ws_buf, L.LORA_DTYPE_F32)
        for j in group:
            got = y[j].cpu().numpy().astype(np.float64)
            assert not np.isfinite(got[~ok]).any()
            # fp32 sums over K and the two-part bf16 operand: 1e-5 of the whole
            assert np.linalg.norm(got[ok] - want[j][ok]) <= 1e-5 * np.linalg.norm(want[j][ok])
