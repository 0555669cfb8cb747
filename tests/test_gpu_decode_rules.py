"""Both sides of the rules that shape a decode call: how far the K range is split and in which steps,
streamed inputs, B kept in the L2 for tall tiles, chunks in flight per wave.  Outputs against the
oracle (sampled rows); the shrink must stay inside the workspace its size query states, also where
that has room for a finer split than the call uses."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
import workloads as W
from gpu_common import check_accumulate, oracle_projection
from harness import DeviceBatch, DevicePool, LayerRunner, bits_from_dev

pytestmark = pytest.mark.gpu

CASES = [
    # rank, h_in, widths, adapters, tokens
    (16, 4096, (392,), 64, 1024),            # eight rows per tile of the bound: four K parts of 32 blocks
    (16, 4096, (392,), 64, 1023),            # one row fewer
    (16, 4096, (392, 136), 64, 300),         # short tiles: eight parts
    (16, 1536, (1032,), 500, 2100),          # too few rows per tile for the coarser split
    (16, 14336, (264,), 24, 700),            # parts of more than two rounds
    (16, 2600, (264,), 100, 1500),           # ragged K, one and a half rounds
    (8, 4160, (520,), 40, 1100),             # rank 8: 64 K values per block
    (32, 4096, (392,), 64, 2048),            # 16 MiB: the streaming limit of ranks 8 to 32, where the batch is sorted first
    (16, 4096, (392,), 300, 2048),           # the same with too many keys to be sorted inside the shrink
    (16, 4096, (392,), 300, 2047),           # just below the limit
    (64, 16384, (264,), 300, 2048),          # 64 MiB: the streaming limit of rank 64
    (64, 4096, (1032,), 40, 1900),           # rank 64: one step in flight, more workgroups
    (64, 1032, (392, 264, 136), 3, 900),     # tall tiles
]


@pytest.mark.parametrize("rank,h_in,widths,n,tokens", CASES)
def test_rules_of_the_decode_kernels(rank, h_in, widths, n, tokens):
    projs = tuple(W.Proj(f"p{i}", h_in, o, "x") for i, o in enumerate(widths))
    w = W.Workload("t", "dense", n, 1, 1, rank, projs, tokens, "zipf", 1.0)
    b = W.make_batch(w, 21, y_mode="normal", no_adapter_frac=0.05, hetero_scale=True)
    ws = W.make_weights(w, 21, bank_elems=1 << 22)
    dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
    run = LayerRunner(dp, db)
    run.v.fill_(float("nan"))
    run.step(0)
    torch.cuda.synchronize()
    assert db.seg.c.tile_rows == 16
    rows = np.sort(np.random.default_rng(21).choice(tokens, min(tokens, 500), replace=False))
    none = b.adapter_id < 0
    for j, p in enumerate(projs):
        full = bits_from_dev(db.y[p.name])
        check_accumulate(np.ascontiguousarray(full[rows]), oracle_projection(b, ws, 0, j, rows=rows),
                         f"decode rules r{rank} {h_in}x{p.h_out}")
        assert np.array_equal(full[none], b.y_in[p.name][none])
    # fp32 output, through a workspace of exactly the stated size between two guards
    x, size, guard = db.inputs["x"], L.lora_v_bytes(dp.pool, 0, tokens), 4096
    buf = torch.full((size + 2 * guard,), 0x5A, dtype=torch.uint8, device="cuda")
    y = torch.zeros(tokens, widths[0], dtype=torch.float32, device="cuda")
    v = buf[guard:guard + size]
    L.lora_shrink(dp.pool, 0, 0, x, x.shape[1], None, db.seg, v)
    L.lora_expand(dp.pool, 0, 0, v, db.seg, y, y.shape[1], L.LORA_DTYPE_F32)
    torch.cuda.synchronize()
    assert bool((buf[:guard] == 0x5A).all()) and bool((buf[guard + size:] == 0x5A).all())
    want = oracle_projection(b, ws, 0, 0, rows=rows, use_y=False).delta
    got = y.cpu().numpy()[rows].astype(np.float64)
    # fp32 accumulation over K and the two-part bf16 operand: 1e-5 of the result's norm
    assert np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want)


def test_a_smaller_batch_may_need_a_larger_workspace():
    """1327 rows over 64 adapters at rank 64 are cut into more K parts than 1328: the size query says so,
    and a call that is handed the larger batch's workspace is refused, not run past its end."""
    desc = L.PoolDesc(64, 1, 1, [(4096, 8)], 64)
    slab = torch.zeros(L.lora_pool_bytes(desc), dtype=torch.uint8, device="cuda")
    pool = L.lora_register_pool(desc, slab)
    P = 1327
    small, large = L.lora_group_ws_bytes(pool, 0, 1, P), L.lora_group_ws_bytes(pool, 0, 1, P + 1)
    assert small > large
    seg, aid = L.Segments(P), torch.zeros(P, dtype=torch.int32, device="cuda")
    x, y = torch.zeros(P, 4096, dtype=torch.bfloat16, device="cuda"), torch.ones(P, 8, dtype=torch.bfloat16, device="cuda")
    L.lora_build_segments(pool, aid, None, P, seg)
    with pytest.raises(L.LoraError) as e:
        L.lora_apply_group(pool, 0, 0, x, 4096, None, seg, [y], [8], torch.empty(large, dtype=torch.uint8, device="cuda"))
    assert e.value.status == -4
    L.lora_apply_group(pool, 0, 0, x, 4096, None, seg, [y], [8], torch.empty(small, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert bool((y == 1).all())
