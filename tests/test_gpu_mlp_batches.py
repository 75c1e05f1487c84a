"""The ladder network at the batch sizes where its kernels change shape: tiles
of 1, 2, 4 and 8 samples (256, 512 and 1024 samples), rounds of 128 samples
in the weight gradients, rows of 8 samples in loss and decode.

Tolerances.  FP32: every sum has at most n = max(128, batch) terms, so a
result is within n * 2^-24 of the sum of its terms' magnitudes; relative to
the largest entry that is below 1e-5 for the outputs (128 terms) and, for the
gradients, below 1e-5 too as long as the rounding errors of the batch's terms
do not all have one sign.  BF16: operands may round to the other neighbour
where the two sides straddle a boundary: 1e-2, as in the network's own test.
"""
import numpy as np
import pytest

from oracle import mlp as omlp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import ladder, qsg  # noqa: E402


def _rel(a, b):
    return np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-30)


@pytest.mark.parametrize("bf16,tol", [(False, 1e-5), (True, 1e-2)])
@pytest.mark.parametrize("B", [1, 2, 127, 128, 129, 255, 257, 511, 513, 1023, 1025, 2050])
def test_batches_match_oracle(B, bf16, tol):
    print(f"[mlp] B={B} bf16={bf16}", flush=True)
    rng = np.random.default_rng(B)
    X = rng.normal(size=(B, 6)).astype(np.float32)
    t = rng.random((B, 31)) + 0.02
    t = (t / t.sum(axis=1, keepdims=True)).astype(np.float32)
    log_l = rng.normal(size=B).astype(np.float32)
    p = ladder.init_params(4).astype(np.float64)
    p[-32:] += 0.2
    p = p.astype(np.float32).astype(np.float64)
    net = ladder.LadderMLP(bf16=bf16, params=p)
    x = torch.tensor(X, device="cuda")
    out, ws = net.forward(x)
    cache = omlp.forward(p, X.astype(np.float64), bf16=bf16)
    assert _rel(out.cpu().numpy(), cache["out"]) < tol
    z = cache["out"].astype(np.float32)
    dz = torch.empty((B, 32), device="cuda")
    loss = torch.empty(B, device="cuda")
    qsg.qsg_mlp_loss(torch.tensor(z, device="cuda"), torch.tensor(t, device="cuda"),
                     torch.tensor(log_l, device="cuda"), dz, loss)
    oloss, odz = omlp.loss_and_grad(z.astype(np.float64), t.astype(np.float64),
                                    log_l.astype(np.float64))
    assert abs(float(loss.double().mean()) - oloss) / abs(oloss) < 1e-5
    assert _rel(dz.cpu().numpy(), odz) < 1e-5
    dz_in = odz.astype(np.float32)
    grads = torch.full((net.n_params,), float("nan"), device="cuda")
    scratch = torch.empty(2 * B * 128, device="cuda")
    qsg.qsg_mlp_backward(net.params, net.bf16, x, ws, torch.tensor(dz_in, device="cuda"), grads,
                         scratch)
    og = omlp.backward(p, cache, dz_in.astype(np.float64), bf16=bf16)
    g, off = grads.cpu().numpy(), 0
    for k, n in omlp.SIZES:
        for size in (k * n, n):
            assert _rel(g[off:off + size], og[off:off + size]) < tol, (k, n, size)
            off += size


@pytest.mark.parametrize("B", [1, 7, 8, 9, 300])
def test_decode_batches_match_oracle(B):
    rng = np.random.default_rng(100 + B)
    z = rng.normal(scale=3.0, size=(B, 32)).astype(np.float32)
    z[0, 1:31] = -300.0  # all of the range in the first gap
    lo, hi = rng.uniform(0.5, 2.0, B), rng.uniform(3.0, 6.0, B)
    lad = torch.empty((B, 32), dtype=torch.float64, device="cuda")
    acc = torch.empty(B, device="cuda")
    qsg.qsg_mlp_decode(torch.tensor(z, device="cuda"), torch.tensor(lo, device="cuda"),
                       torch.tensor(hi, device="cuda"), lad, acc)
    got = lad.cpu().numpy()
    assert np.max(np.abs(got / omlp.decode(z.astype(np.float64), lo, hi) - 1.0)) < 1e-12
    assert np.all(np.diff(got, axis=1) >= 0)
    assert np.array_equal(got[:, 0], lo) and np.array_equal(got[:, -1], hi)
