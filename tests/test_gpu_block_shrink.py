"""The long-segment shrink over blocks of one segment, whose x and A go straight into LDS a stage (64 K values) or two
ahead: K ranges of one to thirteen stages, ranges that end inside one and inside a K-block, with anything
behind the end of a row, and rows with infinities and NaN, which must stay in their own rows."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
import workloads as W
from gpu_common import check_delta, oracle_projection
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


@pytest.mark.parametrize("rank", [16, 32, 64])                                    # one and two stages of A ahead
@pytest.mark.parametrize("h_in", [264, 328, 392, 456, 520, 808])
def test_many_stages_of_one_part(rank, h_in):
    """16416 rows of 8 requests, 129 fours of tiles and more: three K parts at most, which are of 4, 8 or 12 K-blocks for these
    widths; 65536 rows: one part, the whole width of five to thirteen stages."""
    for tokens, most in ((16416, 3), (65536, 1)):
        n = 8
        projs = (W.Proj("gate", h_in, 8, "x"), W.Proj("up", h_in, 8, "x"), W.Proj("down", 8, h_in, "mid"))
        w = W.Workload("t", "moe", n, 1, 1, rank, projs, tokens, "uniform")
        kblocks = -(-h_in // 32)
        most = min(most, kblocks // 4)                                            # no part of less than four K-blocks
        per_part = -(-kblocks // most) + 3 & ~3                                   # whole fours of them
        parts = -(-kblocks // per_part)
        b = W.make_batch(w, 4, y_mode="zero")
        b.adapter_id[:] = np.sort(np.random.default_rng(4).integers(0, n, tokens)).astype(np.int32)
        ws = W.make_weights(w, 4, bank_elems=1 << 20)
        dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
        L.lora_build_segments(dp.pool, db.adapter_id, db.expert_id, tokens, db.seg)
        assert db.seg.c.tile_rows == 32
        bad = [5, tokens - 1]
        xd = torch.full((tokens, h_in + 64), 0x7FC0, dtype=db.inputs["x"].dtype, device="cuda")
        xd[:, :h_in] = db.inputs["x"]
        xd[bad[0], h_in - 1] = 0x7F80
        xd[bad[1], 0] = 0x7FC0
        scratch = torch.full((L.lora_moe_ws_bytes(dp.pool, tokens),), 0xFF, dtype=torch.uint8, device="cuda")
        L.lora_moe_shrink(dp.pool, 0, L.LORA_MOE_UPGATE, xd, xd.shape[1], db.token_of_pair, db.seg, scratch)
        torch.cuda.synchronize()
        v = scratch.view(torch.float32)
        one = tokens * rank
        # a slice starts with its parts; what no part wrote keeps the pattern, which is a NaN
        first = v[:(parts + 1) * one].view(torch.int32) != -1
        assert bool(first[:parts * one].all()) and not bool(first[parts * one:(parts + 1) * one].all())
        y = [torch.zeros(tokens, 8, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        L.lora_moe_expand(dp.pool, 0, L.LORA_MOE_UPGATE, db.seg, y[0], y[1], 8, scratch)
        rows = np.unique(np.concatenate([np.random.default_rng(1).choice(tokens, 300, replace=False), [0, 4, 6, tokens - 2]]))
        rows = rows[~np.isin(rows, bad)]
        for j in range(2):
            got = y[j].float().cpu().numpy().astype(np.float64)
            assert not np.isfinite(got[bad]).any()
            assert np.isfinite(np.delete(got, bad, 0)).all()
            check_delta(got[rows], oracle_projection(b, ws, 0, j, rows=rows, use_y=False).delta, f"stages r{rank} h{h_in}")
