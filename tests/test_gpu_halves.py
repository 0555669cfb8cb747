"""Rank-16 batches whose 32-row tiles run on the decode kernels, in halves: every form those kernels
have (read-modify-write and write-only, bf16 and fp32, gathered rows, one to three projections, K split and
a wave per tile, streamed activations) and both sides of the rule that picks them, against the oracle.
The number of launches tells which kernels a batch runs on (no operand images on the decode kernels)."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
import workloads as W
from gpu_common import check_accumulate, check_delta, oracle_projection
from harness import DeviceBatch, DevicePool, LayerRunner, bits_from_dev
from test_gpu_combine import check_combined, moe_workload, run_combine

pytestmark = pytest.mark.gpu


def on_halves(dp, db, proj0, n):
    return db.seg.c.tile_rows == 32 and L.lora_group_launches(dp.pool, proj0, n, db.P, db.seg) == 2


def sample(P, seed=1, n=600):
    return np.sort(np.random.default_rng(seed).choice(P, min(P, n), replace=False))


@pytest.mark.parametrize("n,tokens,halves", [(64, 12287, True), (64, 12288, False),       # rows of the batch
                                             (101, 12800, True), (100, 12800, False),     # 128 rows per key
                                             (300, 30000, True)])
def test_both_sides_of_the_rule(n, tokens, halves):
    w = W.Workload("t", "dense", n, 1, 1, 16, (W.Proj("p", 264, 136, "x"), W.Proj("q", 264, 72, "x")), tokens, "zipf", 0.6)
    b = W.make_batch(w, 41, y_mode="normal", no_adapter_frac=0.02, hetero_scale=True)
    ws = W.make_weights(w, 41, bank_elems=1 << 22)
    dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
    run = LayerRunner(dp, db)
    run.v.fill_(float("nan"))
    run.step(0)
    torch.cuda.synchronize()
    assert db.seg.c.tile_rows == 32 and on_halves(dp, db, 0, 2) == halves
    rows, none = sample(tokens), b.adapter_id < 0
    for j, p in enumerate(w.projs):
        full = bits_from_dev(db.y[p.name])
        check_accumulate(np.ascontiguousarray(full[rows]), oracle_projection(b, ws, 0, j, rows=rows), f"rule {n} {tokens}")
        assert np.array_equal(full[none], b.y_in[p.name][none])


@pytest.mark.parametrize("policy", [L.LORA_ACT_AUTO, L.LORA_ACT_STREAMING])
@pytest.mark.parametrize("h_in,tokens,n", [(1032, 8200, 40), (72, 44800, 1400)], ids=["K split", "a wave per tile"])
def test_three_projections_and_fp32_outputs(h_in, tokens, n, policy):
    """tile bound of the second case: 1400 + 44800 / 16 = 4200, and a short K range: one wave per tile"""
    projs = tuple(W.Proj(f"p{j}", h_in, o, "x") for j, o in enumerate((136, 264, 8)))
    w = W.Workload("t", "dense", n, 1, 1, 16, projs, tokens, "zipf", 0.4)
    b = W.make_batch(w, 42, y_mode="normal", no_adapter_frac=0.02, hetero_scale=True)
    ws = W.make_weights(w, 42, bank_elems=1 << 22)
    dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
    L.lora_pool_set_activation_policy(dp.pool, policy)
    run = LayerRunner(dp, db)
    run.v.fill_(float("nan"))
    run.step(0)
    torch.cuda.synchronize()
    assert on_halves(dp, db, 0, 3)
    rows = sample(tokens)
    for j, p in enumerate(projs):
        check_accumulate(np.ascontiguousarray(bits_from_dev(db.y[p.name])[rows]),
                         oracle_projection(b, ws, 0, j, rows=rows), f"halves {h_in} {p.name}")
    x = db.inputs["x"]
    src = np.random.default_rng(2).integers(0, tokens, tokens).astype(np.int32)
    y = torch.full((tokens, 264), 0.5, dtype=torch.float32, device="cuda")
    run.v.fill_(float("nan"))
    L.lora_apply(dp.pool, 0, 1, x, h_in, torch.from_numpy(src).cuda(), db.seg, y, 264, run.v, L.LORA_DTYPE_F32)
    torch.cuda.synchronize()
    b.token_of_pair = src
    res = oracle_projection(b, ws, 0, 1, rows=rows, use_y=False)
    got = y.cpu().numpy()[rows].astype(np.float64) - 0.5
    # fp32 sums over K and the two-part bf16 operand, 1e-5 of the result's norm, and the rounding of the
    # addition to 0.5: at most half a unit in the last place of values below 1 (2^-24 sqrt(3)^-1 on average)
    assert np.linalg.norm(got - res.delta) <= 1e-5 * np.linalg.norm(res.delta) + 2.0 ** -24 * np.sqrt(got.size)
    assert torch.equal(y[torch.from_numpy(b.adapter_id < 0).cuda()].cpu(), torch.full((int((b.adapter_id < 0).sum()), 264), 0.5))


@pytest.mark.parametrize("y_mode", ["zero", "normal"])
def test_moe_gate_up_and_combine(y_mode):
    """32 keys, 8200 pairs: gate and up read gathered token rows; the combine's expand writes its pair
    rows without reading them (they hold NaN patterns before)."""
    w = moe_workload(16, 264, 392, n=8, E=4, k=2, tokens=4100)
    r = run_combine(w, 43, y_mode, bad_token=3)
    assert on_halves(r["dp"], r["db"], 2, 1) and on_halves(r["dp"], r["db"], 0, 2)
    check_combined(r, "combine on halves", y_mode)
    b = W.make_batch(w, 44, y_mode=y_mode, hetero_scale=True)
    ws = W.make_weights(w, 44, bank_elems=1 << 22)
    dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
    LayerRunner(dp, db).step(0)
    torch.cuda.synchronize()
    rows = sample(db.P)
    for j, p in enumerate(w.projs):
        res = oracle_projection(b, ws, 0, j, rows=rows)
        got = np.ascontiguousarray(bits_from_dev(db.y[p.name])[rows])
        if y_mode == "zero":
            check_delta(W.bf16_bits_to_f32(got).astype(np.float64), res.delta, f"moe on halves {p.name}")
        else:
            check_accumulate(got, res, f"moe on halves {p.name}")
