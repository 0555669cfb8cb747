"""bench.py's count of a step's kernel launches with the routing-weighted combine: which kernels a batch
runs on decides, not the height of its tiles."""
from types import SimpleNamespace

import pytest

import bench
import paper_2604_07173_amd as L


@pytest.mark.parametrize("tile_rows,group,want", [(16, 2, 1 + 2 + 3), (16, 1, 1 + 1 + 3),
                                                  (32, 2, 1 + 2 + 3),           # rank 16: tiles in halves
                                                  (32, 3, 1 + 3 + 5)])          # images and cleared pair rows
def test_launches_of_a_step_with_the_combine(tile_rows, group, want, monkeypatch):
    monkeypatch.setattr(L, "lora_segments_launches", lambda pool, P: 1)
    monkeypatch.setattr(L, "lora_group_launches", lambda pool, j, n, P, seg, out_dtype=0: group)
    db = SimpleNamespace(P=8, seg=SimpleNamespace(c=SimpleNamespace(tile_rows=tile_rows)))
    w = SimpleNamespace(kind="moe")
    assert bench.launches_per_step(w, SimpleNamespace(pool=None), db, None, combine=True) == want
