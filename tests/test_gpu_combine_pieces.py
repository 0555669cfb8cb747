"""The combine's waves: widths around the 512 columns of one, every number of pair rows that its forms fetch and one
more, numbers of waves that do not fill a workgroup, tokens of which some or all pairs are left out."""
import numpy as np
import pytest

from test_gpu_combine import check_combined, moe_workload, run_combine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h", [8, 504, 512, 520, 1032])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 16])
def test_edges_of_the_pieces(h, k):
    w = moe_workload(rank=8, h=h, f=72, n=5, E=16, k=k, tokens=13)
    r = run_combine(w, 7 + k, "normal", drop=0.4, bad_token=2)
    check_combined(r, f"pieces {h} {k}", "normal")
    on = (r["aid"] >= 0).reshape(w.tokens, k)
    assert np.array_equal(r["got"][~on.any(1)], r["y_tok"][~on.any(1)])
