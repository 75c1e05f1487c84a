"""Correlation sums of sector vectors at every slice size (one part-filled
tile, one tile per block, eight tiles per block): a vector scaled by a power
of two has the same correlations bit for bit (every sum is scaled exactly, up
to norms whose squares come near the ends of the float64 range), an estimate
from twice the same vector is that vector's own result, and a state of one
configuration pair is fully correlated."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402


@pytest.mark.parametrize("L", [2, 3, 4, 5])
def test_scaling_and_closed_forms(L):
    print(f"[corr] L={L}", flush=True)
    n = qsg.tm_dim(L)
    g = torch.Generator(device="cuda").manual_seed(L)
    v = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    want = qsg.tm_correlations(L, v)
    for scale in (2.0 ** 450, 2.0 ** -450):
        assert qsg.tm_correlations(L, scale * v) == want
    for r in qsg.tm_correlations_lt(L, v, 2.0 * v, 3.0, 2.0, [0, 1, 7]):
        # (a + b)^2 = 1 up to the rounding of the three products
        for k in ("Q2", "Q4", "F"):
            assert abs(r[k] - want[k]) <= 1e-14 * want["Q4"], (k, r, want)
    one = torch.zeros_like(v)
    one[n // 3] = -2.5
    V = float(L * L)
    r = qsg.tm_correlations(L, one)
    assert r["Q2"] == V ** 2 and r["Q4"] == V ** 4
    assert abs(r["F"]) <= 1e-12 * V * V  # the cosines of a full row sum to 0
