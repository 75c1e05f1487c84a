"""The ladder network's kernels on unusual values: results equal those of the
formulas taken one sample (or one logit) after the other."""
import numpy as np
import pytest

from oracle import mlp as omlp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402


def _decode(z, lo, hi):
    B = len(z)
    lad = torch.empty((B, 32), dtype=torch.float64, device="cuda")
    acc = torch.empty(B, device="cuda")
    qsg.qsg_mlp_decode(torch.tensor(z, device="cuda"), torch.tensor(lo, device="cuda"),
                       torch.tensor(hi, device="cuda"), lad, acc)
    return lad.cpu().numpy()


def _walk(z, lo, hi):
    """The points one after the other: never below the one before, the last
    inner point not above the end."""
    out = omlp.decode(z.astype(np.float64), lo, hi)
    out[:, 0] = lo
    for i in range(1, 31):
        out[:, i] = np.maximum(out[:, i], out[:, i - 1])
    out[:, 30] = np.minimum(out[:, 30], hi)
    out[:, 31] = hi
    return out


def test_decode_of_ends_in_either_order():
    rng = np.random.default_rng(8)
    z = rng.normal(scale=2.0, size=(11, 32)).astype(np.float32)
    lo = rng.uniform(1.0, 4.0, 11)
    hi = lo * np.where(np.arange(11) % 3 == 0, 1.7, np.where(np.arange(11) % 3 == 1, 0.6, 1.0))
    got, want = _decode(z, lo, hi), _walk(z, lo, hi)
    # exponentials and logarithms of either side are good to a few 2^-53
    assert np.max(np.abs(got / want - 1.0)) < 1e-12
    back = lo > hi
    assert np.array_equal(got[back, 1:30], np.repeat(lo[back, None], 29, axis=1))
    assert np.array_equal(got[:, 31], hi)
