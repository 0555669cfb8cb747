"""Work items of the long-segment shrink (blocks of 128 rows of one segment, looked up in the segment
list) and the decode kernels on the halves of 32-row tiles: segment lengths around the block, tile and
half sizes, more segments than one look-up pass covers, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
import workloads as W
from gpu_common import check_accumulate, check_delta, oracle_projection
from harness import DeviceBatch, DevicePool, LayerRunner, bits_from_dev

pytestmark = pytest.mark.gpu


def run_lengths(lengths, rank, widths, h_in, seed, y_mode, shuffle, n=None):
    n = n or len(lengths)
    aid = np.repeat(np.arange(len(lengths), dtype=np.int32), lengths)
    aid = np.concatenate([aid, np.full(5, -1, np.int32)])
    if shuffle:
        aid = np.random.default_rng(seed).permutation(aid)
    projs = tuple(W.Proj(f"p{i}", h_in, o, "x") for i, o in enumerate(widths))
    w = W.Workload("t", "dense", n, 1, 1, rank, projs, aid.size, "uniform")
    b = W.make_batch(w, seed, y_mode=y_mode, hetero_scale=True)
    b.adapter_id[:] = aid
    ws = W.make_weights(w, seed, bank_elems=1 << 22)
    dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
    run = LayerRunner(dp, db)
    run.v.fill_(float("nan"))                  # nothing may depend on what the workspace holds
    run.step(0)
    torch.cuda.synchronize()
    assert db.seg.c.tile_rows == 32
    rows = np.sort(np.random.default_rng(seed).choice(aid.size, min(aid.size, 700), replace=False))
    none = b.adapter_id < 0
    for j, p in enumerate(projs):
        res = oracle_projection(b, ws, 0, j, rows=rows)
        full = bits_from_dev(db.y[p.name])
        got = np.ascontiguousarray(full[rows])
        if y_mode == "zero":
            check_delta(W.bf16_bits_to_f32(got).astype(np.float64), res.delta, f"blocks r{rank} {p.name}")
        else:
            check_accumulate(got, res, f"blocks r{rank} {p.name}")
        assert np.array_equal(full[none], b.y_in[p.name][none])
    return dp, db


EDGES = [1, 127, 128, 129, 0, 31, 32, 33, 255, 256, 257, 16, 17, 384]


@pytest.mark.parametrize("rank", [16, 32, 64])
@pytest.mark.parametrize("lengths,shuffle", [(EDGES, True), ([1], False), ([2 + i % 3 for i in range(600)], True),
                                             ([0] * 255 + [130, 3, 200], False)])
def test_blocks_of_segments(rank, lengths, shuffle, monkeypatch):
    monkeypatch.setenv("LORA_TILE_ROWS", "32")
    run_lengths(lengths, rank, (392, 136, 264), 1032, 3, "normal", shuffle)


@pytest.mark.parametrize("rank", [32, 64])
@pytest.mark.parametrize("lengths,h_in,parts", [([2048] * 8, 2048, 4), ([2047] * 7 + [2055], 2048, 3),
                                                ([1024] * 8, 2048, 8), ([400] * 12, 2048, 4), ([8192] * 16, 512, 1)])
def test_k_parts_follow_the_tiles_of_the_batch(lengths, h_in, parts, rank):
    """Fours of 32-row tiles on 512 places (220 below 64 fours): equal requests of 2048 rows have 128
    fours and take four K parts, and one tile more takes three, though the number of rows is the same.
    Every row of every part is written, and no other."""
    n, P = len(lengths), sum(lengths)
    w = W.Workload("t", "dense", n, 1, 1, rank, (W.Proj("p", h_in, 8, "x"),), P, "uniform")
    b = W.make_batch(w, 6, y_mode="zero")
    b.adapter_id[:] = np.repeat(np.arange(n, dtype=np.int32), lengths)
    dp, db = DevicePool(W.make_weights(w, 6, bank_elems=1 << 22), b.scale), DeviceBatch(b)
    run = LayerRunner(dp, db)
    run.build_segments()
    run.v.fill_(float("nan"))
    x = db.inputs["x"]
    L.lora_shrink(dp.pool, 0, 0, x, x.shape[1], None, db.seg, run.v)
    torch.cuda.synchronize()
    assert db.seg.c.tile_rows == 32
    written = ~torch.isnan(run.v)
    assert int(written.sum()) == parts * P * rank and bool(written[:parts * P * rank].all())


@pytest.mark.parametrize("rank,n_proj", [(16, 1), (16, 2), (32, 1), (32, 2), (64, 1), (64, 3)])
@pytest.mark.parametrize("n", [64, 65, 129, 4096, 4097])
def test_both_ways_to_number_the_work_items(n, rank, n_proj, monkeypatch):
    """Blocks of one segment (launches of two projections, up to 4096 segments) and groups of four tiles:
    short and long segments mixed, every group of tiles with a segment boundary and, in the run of 513
    rows, some without."""
    monkeypatch.setenv("LORA_TILE_ROWS", "32")
    lengths = [1 + (i * 7) % 3 for i in range(n)]
    lengths[n // 3], lengths[n // 2], lengths[-1] = 513, 130, 33
    run_lengths(lengths, rank, (136, 40, 8)[:n_proj], 392, 5, "normal", True)


def test_finding_a_work_items_segment_is_cheap():
    """The gate/up shrink of the same 524288 rows in 64 and in 16384 segments.  The many short ones read 256
    times the weights; walking over the list of segments for every work item cost far more than that (1.5
    times the time of the few long ones; 7.9 times with the walk)."""
    P, h_in, us = 524288, 64, {}
    for n in (64, 16384):
        projs = (W.Proj("gate", h_in, 8, "x"), W.Proj("up", h_in, 8, "x"), W.Proj("down", 8, h_in, "mid"))
        w = W.Workload("t", "moe", n, 1, 1, 32, projs, P, "uniform")
        b = W.make_batch(w, 7, y_mode="zero")
        dp, db = DevicePool(W.make_weights(w, 7, bank_elems=1 << 20), b.scale), DeviceBatch(b)
        run = LayerRunner(dp, db)
        run.build_segments()
        assert db.seg.c.tile_rows == 32
        x, times = db.inputs["x"], []
        for _ in range(15):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            L.lora_moe_shrink(dp.pool, 0, L.LORA_MOE_UPGATE, x, h_in, db.token_of_pair, db.seg, run.ws)
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 1e3)
        us[n] = sorted(times)[len(times) // 2]
    print("us by segments:", us)
    assert us[16384] <= 4 * us[64], us


@pytest.mark.parametrize("y_mode", ["zero", "normal"])
@pytest.mark.parametrize("lengths", [EDGES * 5, [8187], [104 + 3 * i for i in range(48)]])
def test_halves_of_tiles_at_rank_16(lengths, y_mode):
    """8192 to 12287 rows at rank 16: 32-row tiles on the decode kernels, which take them in halves."""
    dp, db = run_lengths(lengths, 16, (392, 264), 520, 4, y_mode, True)
    assert 8192 <= db.P < 12288
    assert L.lora_group_launches(dp.pool, 0, 2, db.P, db.seg) == 2
