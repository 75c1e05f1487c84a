"""The ladder network's kernels on unusual values and on batches where loss and
decode give a sample one thread: results equal those of the formulas taken one
sample (or one logit) after the other."""
import numpy as np
import pytest

from oracle import mlp as omlp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import ladder, qsg  # noqa: E402


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


def _kind(a):
    """0 finite, 1 NaN, 2 inf, 3 -inf."""
    return np.where(np.isnan(a), 1, np.where(np.isposinf(a), 2, np.where(np.isneginf(a), 3, 0)))


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("B", [3, 128, 131])
def test_an_infinite_weight_reaches_the_gradients_it_meets(B, bf16):
    """The weight gradients are formed 128 samples at a time; the places of a
    round without a sample add nothing, whatever the weights hold."""
    print(f"[mlp] B={B} bf16={bf16}", flush=True)
    rng = np.random.default_rng(B)
    X = rng.normal(size=(B, 6)).astype(np.float32)
    p = ladder.init_params(4).astype(np.float32)
    out_w = len(p) - 32 - 128 * 32
    p[out_w + 7 * 32 + 3] = np.inf
    p[out_w - 128 + 7] = 12.0  # its unit is on for every sample: one sign of infinity
    dout = rng.uniform(0.5, 1.5, size=(B, 32)).astype(np.float32)
    net = ladder.LadderMLP(bf16=bf16, params=p.astype(np.float64))
    x = torch.tensor(X, device="cuda")
    _, ws = net.forward(x)
    grads = torch.empty(net.n_params, device="cuda")
    qsg.qsg_mlp_backward(net.params, net.bf16, x, ws, torch.tensor(dout, device="cuda"), grads,
                         torch.empty(2 * B * 128, device="cuda"))
    p = p.astype(np.float64)
    with np.errstate(invalid="ignore"):
        cache = omlp.forward(p, X.astype(np.float64), bf16=bf16)
        # the activations of the pass itself: far below zero an FP32 one is 0,
        # and 0 times infinity no infinity
        for l, act in enumerate(ws.cpu().numpy()[:6 * B * 128].reshape(3, 2, B, 128)[:, 1]):
            cache["inputs"][l + 1] = omlp.to_bf16(act) if bf16 else act.astype(np.float64)
        want = omlp.backward(p, cache, dout.astype(np.float64), bf16=bf16)
    got = _kind(grads.cpu().numpy())
    assert np.array_equal(got, _kind(want)), np.nonzero(got != _kind(want))[0][:8]
    assert np.any(_kind(want) == 2)


def _large_batch(B):
    rng = np.random.default_rng(B)
    z = rng.normal(scale=2.0, size=(B, 32)).astype(np.float32)
    t = rng.random((B, 31)) + 0.02
    t[::5, 3:9] = 0.0
    t = (t / t.sum(axis=1, keepdims=True)).astype(np.float32)
    z[1, 4], z[2, 0], t[3, 2], z[4, :31] = np.nan, np.inf, np.nan, -np.inf
    lo = rng.uniform(0.5, 2.0, B)
    hi = lo * np.where(np.arange(B) % 7 == 0, 0.5, rng.uniform(1.0, 3.0, B))
    lo[5], hi[6] = np.nan, np.nan
    return z, t, rng.normal(size=B).astype(np.float32), lo, hi


def _loss(z, t, log_l):
    dz, loss = torch.empty((len(z), 32), device="cuda"), torch.empty(len(z), device="cuda")
    qsg.qsg_mlp_loss(*(torch.tensor(a, device="cuda") for a in (z, t, log_l)), dz, loss)
    return loss.cpu().numpy(), dz.cpu().numpy()


@pytest.mark.parametrize("B", [8193, 16384 + 63])
def test_loss_and_decode_of_large_batches_are_those_of_their_parts(B):
    """8192 samples are the most that take 32 threads each.  Losses and
    ladders of a batch are those of its halves bit for bit; the gradients too,
    up to the rounding of 1/B and of its product (2^-24 each)."""
    print(f"[mlp] B={B}", flush=True)
    z, t, log_l, lo, hi = _large_batch(B)
    loss, dz = _loss(z, t, log_l)
    lad = _decode(z, lo, hi)
    cuts = [(i, min(i + 4096, B)) for i in range(0, B, 4096)]
    parts = [_loss(z[i:j], t[i:j], log_l[i:j]) for i, j in cuts]
    assert np.array_equal(loss, np.concatenate([p[0] for p in parts]), equal_nan=True)
    scaled = np.concatenate([p[1].astype(np.float64) * (j - i) / B for p, (i, j) in zip(parts, cuts)])
    assert np.array_equal(np.isnan(dz), np.isnan(scaled))
    assert np.nanmax(np.abs(dz - scaled) / np.maximum(np.abs(scaled), 1e-30)) < 4 * 2.0 ** -24
    assert np.array_equal(lad, np.concatenate([_decode(z[i:j], lo[i:j], hi[i:j]) for i, j in cuts]),
                          equal_nan=True)
