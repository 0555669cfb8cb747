"""Order of the wave items of the long-segment expand: runs of four tiles for narrow fp32 outputs (up to 2048 columns in all) and for
bf16 rows of 4 KiB that a call covers whole, chunks first otherwise; numbers of tiles that leave the last run and the last pair of tiles unfinished."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
import workloads as W
from gpu_common import check_delta, oracle_projection
from harness import DeviceBatch, DevicePool, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [16, 32, 64])
@pytest.mark.parametrize("widths", [(8,), (136, 40), (2048,), (2056,), (1024, 896, 128), (1024, 896, 136)])
@pytest.mark.parametrize("lengths", [[1], [33, 31], [300, 5, 129], [64] * 8, [513, 0, 1, 95]])
def test_every_tile_and_chunk_once(lengths, widths, rank, monkeypatch):
    monkeypatch.setenv("LORA_TILE_ROWS", "32")
    n, P = len(lengths), sum(lengths)
    projs = tuple(W.Proj(f"p{i}", 72, o, "x") for i, o in enumerate(widths))
    w = W.Workload("t", "dense", n, 1, 1, rank, projs, P, "uniform")
    b = W.make_batch(w, 2, y_mode="normal", hetero_scale=True)
    b.adapter_id[:] = np.random.default_rng(2).permutation(np.repeat(np.arange(n, dtype=np.int32), lengths))
    ws = W.make_weights(w, 2, bank_elems=1 << 20)
    dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
    L.lora_build_segments(dp.pool, to_dev(b.adapter_id), None, P, db.seg)
    assert db.seg.c.tile_rows == 32
    x = db.inputs["x"]
    scratch = torch.full((L.lora_group_ws_bytes(dp.pool, 0, len(projs), P),), 0xFF, dtype=torch.uint8, device="cuda")
    ys = [torch.ones(P, o, dtype=torch.float32, device="cuda") for o in widths]
    L.lora_apply_group(dp.pool, 0, 0, x, x.shape[1], None, db.seg, ys, list(widths), scratch, L.LORA_DTYPE_F32)
    for j, y in enumerate(ys):
        want = oracle_projection(b, ws, 0, j, use_y=False).delta
        got = y.cpu().numpy().astype(np.float64) - 1.0
        # fp32 sums over K, the two-part bf16 operand and the rounding at 1: 2^-24 of it beside deltas of about the scale of 1
        assert np.abs(got - want).max() <= 1e-5 * np.abs(want).max() + 2.0 ** -23, f"projection {j}"


@pytest.mark.parametrize("rank", [16, 32, 64])
@pytest.mark.parametrize("widths,ld", [((2048,), 2048), ((1024, 1024), 2048), ((512, 1024, 512), 2048), ((2040,), 2048), ((1920,), 2048),
                                       ((2048,), 2056), ((2048, 8), 2048)])
@pytest.mark.parametrize("lengths", [[1], [33, 31], [300, 5, 129], [64] * 6, [97] * 2])
def test_every_tile_and_chunk_once_in_bf16(lengths, widths, ld, rank, monkeypatch):
    """Fused outputs beside each other in rows of `ld` columns where they fit; columns behind them stay as they are."""
    monkeypatch.setenv("LORA_TILE_ROWS", "32")
    n, P = len(lengths), sum(lengths)
    projs = tuple(W.Proj(f"p{i}", 72, o, "x") for i, o in enumerate(widths))
    w = W.Workload("t", "dense", n, 1, 1, rank, projs, P, "uniform")
    b = W.make_batch(w, 2, y_mode="zero", hetero_scale=True)
    b.adapter_id[:] = np.random.default_rng(2).permutation(np.repeat(np.arange(n, dtype=np.int32), lengths))
    ws = W.make_weights(w, 2, bank_elems=1 << 20)
    dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
    L.lora_build_segments(dp.pool, to_dev(b.adapter_id), None, P, db.seg)
    assert db.seg.c.tile_rows == 32
    x = db.inputs["x"]
    scratch = torch.full((L.lora_group_ws_bytes(dp.pool, 0, len(projs), P),), 0xFF, dtype=torch.uint8, device="cuda")
    rows, ys, at = [], [], 0
    for o in widths:
        if not rows or at + o > ld:
            rows.append(torch.zeros(P, ld, dtype=torch.bfloat16, device="cuda"))
            at = 0
        ys.append(rows[-1][:, at:at + o])
        at += o
    L.lora_apply_group(dp.pool, 0, 0, x, x.shape[1], None, db.seg, ys, [ld] * len(widths), scratch, L.LORA_DTYPE_BF16)
    for j, y in enumerate(ys):
        check_delta(y.float().cpu().numpy().astype(np.float64), oracle_projection(b, ws, 0, j, use_y=False).delta, f"order r{rank} {widths} {j}")
    assert not rows[-1][:, at:].any()


@pytest.mark.parametrize("dtype,h,rank,most", [(torch.float32, 1024, 16, 1.2), (torch.bfloat16, 2048, 32, 1.07)])
def test_rows_a_power_of_two_apart(dtype, h, rank, most):
    """16384 rows of eight equal requests: rows of 4 KiB take 1.01 of the time of rows of 4.25 KiB; with waves that all start
    with the first rows of a tile and one chunk beside the other 1.35 in fp32 and 1.20 in bf16."""
    n, P = 8, 16384
    out = L.LORA_DTYPE_F32 if dtype == torch.float32 else L.LORA_DTYPE_BF16
    w = W.Workload("t", "dense", n, 1, 1, rank, (W.Proj("p", 64, h, "x"),), P, "uniform")
    b = W.make_batch(w, 2, y_mode="zero")
    ids = to_dev(np.repeat(np.arange(n, dtype=np.int32), P // n))
    dp, seg, us = DevicePool(W.make_weights(w, 2, bank_elems=1 << 20), b.scale), L.Segments(P), {}
    L.lora_build_segments(dp.pool, ids, None, P, seg)
    assert seg.c.tile_rows == 32
    scratch = torch.zeros(L.lora_group_ws_bytes(dp.pool, 0, 1, P), dtype=torch.uint8, device="cuda")
    for ld in (h, h + h // 16):
        y, times = torch.zeros(P, ld, dtype=dtype, device="cuda"), []
        stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.stream(stream):
            L.lora_expand(dp.pool, 0, 0, scratch, seg, y, ld, out)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(20):
                L.lora_expand(dp.pool, 0, 0, scratch, seg, y, ld, out)
        for _ in range(15):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            graph.replay()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 50)
        us[ld] = sorted(times)[7]
    print("us by row stride:", us)
    assert us[h] <= most * us[h + h // 16], us
