"""Repacking of adapters from 16-byte aligned sources (LDS and register transposes) and from sources
at odd addresses (one value at a time): both give the slab that the layout functions define, read
back bit for bit, at ragged widths, at adapter ranks below the pool's and for whole layers and
single units."""
import numpy as np
import pytest
import torch

import paper_2604_07173_amd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank,own", [(8, 8), (8, 3), (16, 16), (16, 5), (32, 32), (32, 24), (64, 64), (64, 33)])
@pytest.mark.parametrize("shapes", [[(8, 8)], [(64, 128), (72, 136)], [(200, 1032), (1032, 200), (40, 24)]])
def test_aligned_and_odd_sources_pack_alike(rank, own, shapes):
    n_experts, slabs = 3, []
    elems = n_experts * sum((i + o) * own for i, o in shapes)
    rng = np.random.default_rng(rank * 100 + own)
    bits = rng.integers(-(1 << 15), 1 << 15, elems, dtype=np.int64).astype(np.int16)
    for shift in (0, 1):                                   # elements: the second source is only 2-byte aligned
        buf = torch.empty(elems + 8, dtype=torch.int16, device="cuda")
        src = buf[shift:shift + elems]
        src.copy_(torch.from_numpy(bits))
        desc = L.PoolDesc(2, 1, n_experts, shapes, rank, adapter_rank=[own, rank])
        slab = torch.zeros(L.lora_pool_bytes(desc), dtype=torch.uint8, device="cuda")
        pool = L.lora_register_pool(desc, slab)
        L.lora_pool_load_adapter_layer(pool, 0, 0, src)
        at = 0
        for e in range(n_experts):
            for j, (i, o) in enumerate(shapes):
                A, B = bits[at:at + i * own].reshape(i, own), bits[at + i * own:at + (i + o) * own].reshape(own, o)
                at += (i + o) * own
                Ao = torch.full((i, rank), 7, dtype=torch.int16, device="cuda")
                Bo = torch.full((rank, o), 7, dtype=torch.int16, device="cuda")
                L.lora_pool_read_unit(pool, 0, 0, e, j, Ao, Bo)
                got_a, got_b = Ao.cpu().numpy(), Bo.cpu().numpy()
                assert np.array_equal(got_a[:, :own], A) and not got_a[:, own:].any(), (e, j)
                assert np.array_equal(got_b[:own], B) and not got_b[own:].any(), (e, j)
        # the units' bytes, behind the table (which holds the slab's own addresses)
        first = min(L.lora_pool_unit_layout(pool, 0, 0, e, j)["A_offset"] for e in range(n_experts)
                    for j in range(len(shapes)))
        slabs.append(slab[first:].clone())
        # single units, from the same source
        slab2 = torch.zeros_like(slab)
        pool2 = L.lora_register_pool(desc, slab2)
        at = 0
        for e in range(n_experts):
            for j, (i, o) in enumerate(shapes):
                L.lora_pool_load_unit(pool2, 0, 0, e, j, src.data_ptr() + 2 * at, src.data_ptr() + 2 * (at + i * own))
                at += (i + o) * own
        torch.cuda.synchronize()
        assert torch.equal(slab2[first:], slabs[-1])
    assert torch.equal(slabs[0], slabs[1])
