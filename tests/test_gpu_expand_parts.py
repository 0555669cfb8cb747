"""The K parts of v that the decode expand adds: one to eight parts (batches of loads, parts dealt over the lanes
of a quad), tiles of every height from one row to a full one and a remainder, every rank and output form."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L
import workloads as W
from gpu_common import check_accumulate, oracle_projection
from harness import DeviceBatch, DevicePool, LayerRunner, bits_from_dev

pytestmark = pytest.mark.gpu

HEIGHTS = list(range(1, 18))             # rows of adapter 0, 1, ...: tiles of 1 .. 16 rows, and 16 + 1


@pytest.mark.parametrize("rank", [8, 16, 32, 64])
@pytest.mark.parametrize("parts", [1, 2, 3, 5, 8])
def test_parts_and_tile_heights(rank, parts):
    h_in = parts * 4 * (64 if rank == 8 else 32)          # four K-blocks a part, as many parts as that gives
    n, tokens = len(HEIGHTS), sum(HEIGHTS)
    projs = (W.Proj("p0", h_in, 264, "x"), W.Proj("p1", h_in, 136, "x"))
    w = W.Workload("t", "dense", n, 1, 1, rank, projs, tokens, "zipf", 1.0)
    b = W.make_batch(w, 5, y_mode="normal", hetero_scale=True)
    b.adapter_id[:] = np.random.default_rng(5).permutation(np.repeat(np.arange(n), HEIGHTS))
    ws = W.make_weights(w, 5, bank_elems=1 << 20)
    dp, db = DevicePool(ws, b.scale), DeviceBatch(b)
    LayerRunner(dp, db).step(0)
    for j, p in enumerate(projs):
        check_accumulate(bits_from_dev(db.y[p.name]), oracle_projection(b, ws, 0, j), f"parts r{rank} x{parts}")
    x, size = db.inputs["x"], L.lora_v_bytes(dp.pool, 0, tokens)
    assert size == -(-parts * tokens * rank * 4 // 256) * 256       # so many parts are what the batch is cut into
    v = torch.full((size // 4,), float("nan"), dtype=torch.float32, device="cuda")
    y = torch.zeros(tokens, 264, dtype=torch.float32, device="cuda")
    L.lora_shrink(dp.pool, 0, 0, x, x.shape[1], None, db.seg, v)
    L.lora_expand(dp.pool, 0, 0, v, db.seg, y, y.shape[1], L.LORA_DTYPE_F32)
    got = y.cpu().numpy().astype(np.float64)
    want = oracle_projection(b, ws, 0, 0, use_y=False).delta
    # v enters the second product as bf16 hi + lo: hi is cut off below 2^-7 of the value, lo is rounded to 2^-9 of
    # what remains, so an entry is off by 2^-16 of itself at most; the fp32 sums over K by about sqrt(K) roundings
    for a in range(n):
        A, B = (W.bf16_bits_to_f32(m).astype(np.float64) for m in ws.unit_arrays(a, 0, 0, 0))
        r = np.nonzero(b.adapter_id == a)[0]
        xa = W.bf16_bits_to_f32(b.inputs["x"][r]).astype(np.float64)
        bound = b.scale[a] * (2.0 ** -16 * np.abs(xa @ A) + 4 * h_in ** 0.5 * 2.0 ** -24 * (np.abs(xa) @ np.abs(A))) @ np.abs(B)
        assert (np.abs(got[r] - want[r]) <= bound).all()


@pytest.mark.parametrize("rank", [8, 16, 32, 64])
@pytest.mark.parametrize("parts", [2, 3, 5, 8])
def test_bits_of_a_row_do_not_depend_on_its_tile(rank, parts):
    """A row's update does not depend on the rows that travel with it: the same row under the same weights has the
    same bits in tiles of every height, whichever lanes fetched its parts of v."""
    h_in, h_out = parts * 4 * (64 if rank == 8 else 32), 264
    n, P = len(HEIGHTS), sum(HEIGHTS)
    g = torch.Generator(device="cuda").manual_seed(rank + parts)
    weights = torch.randn((h_in + h_out) * rank, generator=g, device="cuda").bfloat16()
    desc = L.PoolDesc(n, 1, 1, [(h_in, h_out)], rank, scale=[1.25] * n)
    slab = torch.empty(L.lora_pool_bytes(desc), dtype=torch.uint8, device="cuda")
    pool = L.lora_register_pool(desc, slab)
    for a in range(n):
        L.lora_pool_load_adapter_layer(pool, a, 0, weights)
    aid = torch.from_numpy(np.random.default_rng(7).permutation(np.repeat(np.arange(n), HEIGHTS)).astype(np.int32)).cuda()
    x = torch.randn(1, h_in, generator=g, device="cuda").bfloat16().repeat(P, 1)
    seg = L.Segments(P)
    L.lora_build_segments(pool, aid, None, P, seg)
    size = L.lora_v_bytes(pool, 0, P)
    assert size == -(-parts * P * rank * 4 // 256) * 256
    v = torch.full((size // 4,), float("nan"), dtype=torch.float32, device="cuda")
    y = torch.zeros(P, h_out, dtype=torch.float32, device="cuda")
    L.lora_shrink(pool, 0, 0, x, h_in, None, seg, v)
    L.lora_expand(pool, 0, 0, v, seg, y, h_out, L.LORA_DTYPE_F32)
    assert bool(y[0].any())
    differ = (y != y[0]).any(dim=1).cpu().numpy()
    heights = np.repeat(HEIGHTS, HEIGHTS)[np.argsort(np.argsort(aid.cpu().numpy(), kind="stable"), kind="stable")]
    assert not differ.any(), sorted(set(heights[differ].tolist()))
