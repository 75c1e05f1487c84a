"""Lanczos at the step counts where its kernels change: up to 8, 16, ... 48
basis vectors held in registers (32 in the first dot products), and more.
After m steps the residual of the Ritz pair is beta_m |y_m| exactly, so the
estimate, the Rayleigh quotient and the norm of the returned vector are
checked against the product itself.

Tolerances: a product, a dot product and a norm over 2^15 entries in float64
are good to well under 1e-12 of |T| = theta (the worst-case bound of a sum of
2^15 terms is 2^15 * 2^-53 = 4e-12 of the sum of magnitudes, reached only if
all roundings have one sign)."""
import numpy as np
import pytest

import qsg_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402


@pytest.mark.parametrize("parity", [1, -1])
@pytest.mark.parametrize("steps", [1, 2, 7, 8, 9, 16, 17, 24, 25, 32, 33, 40, 41, 48, 49, 65])
def test_ritz_pair_after_a_number_of_steps(steps, parity):
    print(f"[lanczos] steps={steps} parity={parity}", flush=True)
    # weak space coupling: the spectrum is dense and the steps are not used up
    c = W.transfer_case(L=4, k=0.02, k_perp=1.5, seed=11)
    d = qsg.tm_desc(c.L, c.k, c.k_perp, c.jx, c.jy, parity)
    r = qsg.tm_lanczos(d, steps, 1, 0.0, seed=3, want_vector=True)
    assert r["iters"] <= steps
    v = r["vector"]
    tv = torch.empty_like(v)
    qsg.tm_apply(d, v, tv)
    theta = r["values"][0]
    assert abs(float(v @ v) - 1.0) < 1e-12
    assert abs(float(v @ tv) - theta) < 1e-12 * theta
    assert abs(float((tv - theta * v).norm()) - r["resid"][0]) < 1e-12 * theta
