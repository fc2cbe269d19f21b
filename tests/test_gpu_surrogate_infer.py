"""Surrogate inference in one pass (xbar_sg_infer_bf16) against the layer-by-layer path:
tile edges, maps smaller than a tile, every rounding of the channel count and every depth.

The last map has the same bits in both, so currents and estimates may differ only by the
rounding of float64 sums over at most m rows: relative tolerance 4 m eps (1 + S), with S
the largest mean absolute map value over |1 + yhat| (cancellation in 1 + yhat), plus the
exponential's amplification 2 of the estimate's own sum.
"""
import numpy as np
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth,C", [(2, 1), (2, 32), (3, 7), (3, 16), (4, 8), (4, 20), (4, 32), (5, 17), (5, 32)])
@pytest.mark.parametrize("B,m,n", [(1, 1, 1), (3, 7, 33), (2, 8, 32), (5, 17, 100), (2, 40, 65), (64, 128, 128)])
def test_one_pass_inference_matches_layers(B, m, n, depth, C):
    import torch

    from paper_2410_19993_amd import _lib
    from paper_2410_19993_amd.surrogate import Surrogate
    rng = np.random.default_rng(1000 * depth + 10 * C + m + n)
    log(f"case infer B={B} {m}x{n} depth={depth} C={C}")
    G = torch.from_numpy(np.exp(rng.uniform(np.log(1e-6), np.log(1e-4), (B, m, n)))).cuda()
    V = torch.from_numpy(rng.uniform(0.0, 0.5, (B, m))).cuda()
    r = torch.from_numpy(rng.uniform(1.0, 5.0, B)).cuda()
    net = Surrogate(channels=C, seed=3, depth=depth, zero_last=False)
    net.params += 0.01 * torch.from_numpy(rng.normal(size=net.params.numel()).astype(np.float32)).cuda()
    assert _lib.xbar_sg_infer_workspace_bytes(B, m, n, C, depth) > 0
    est = torch.empty((B, n), dtype=torch.float64, device="cuda")
    I = net.predict(G, V, r, est=est).cpu().numpy()
    est = est.cpu().numpy()
    Y = net.forward(G, V, r)
    I2 = torch.empty((B, n), dtype=torch.float64, device="cuda")
    e2 = torch.empty_like(I2)
    _lib.xbar_sg_predict(B, m, n, Y, G, V, I2, e2, net._stream())
    I2, e2 = I2.cpu().numpy(), e2.cpu().numpy()
    Yh = Y.cpu().numpy().astype(np.float64)
    one = np.abs(1.0 + Yh[:, 0].mean(axis=1))
    S = np.abs(Yh).mean(axis=2).max(axis=1) / one
    tol = 4 * m * np.finfo(float).eps * (1 + S)
    assert np.all(np.abs(I - I2) <= tol * np.abs(I2) + 1e-300)
    assert np.all(np.abs(est - e2) <= 2 * (tol + 4 * m * np.finfo(float).eps * np.abs(Yh).mean(axis=2).max(axis=1)) * e2)


def test_sizes_outside_the_one_pass_call():
    from paper_2410_19993_amd import _lib
    for args in ((1, 8, 8, 8, 6), (1, 8, 8, 33, 4), (1, 2049, 8, 8, 4), (0, 8, 8, 8, 4), (1, 8, 8, 8, 1)):
        assert _lib.xbar_sg_infer_workspace_bytes(*args) == -1


@pytest.mark.parametrize("which", ["out_on_r", "est_on_r", "est_on_V"])
def test_outputs_on_inputs_that_are_read_before_them(which):
    """Outputs in the place of an input that the currents' last step does not read (the
    resistances, or for the estimates the input vectors) are taken, and are what separate
    buffers receive; currents on G or V are refused."""
    import torch

    from paper_2410_19993_amd import _lib
    from paper_2410_19993_amd.surrogate import Surrogate
    rng = np.random.default_rng(7)
    B, m, n = (5, 33, 33) if which == "est_on_V" else (5, 33, 1)
    log(f"case infer {which}")
    G = torch.from_numpy(np.exp(rng.uniform(np.log(1e-6), np.log(1e-4), (B, m, n)))).cuda()
    V = torch.from_numpy(rng.uniform(0.0, 0.5, (B, m))).cuda()
    r = torch.from_numpy(rng.uniform(1.0, 5.0, B)).cuda()
    net = Surrogate(channels=8, seed=3, depth=3, zero_last=False)
    e0 = torch.empty((B, n), dtype=torch.float64, device="cuda")
    I0 = net.predict(G, V, r, est=e0)
    out = r.view(B, 1) if which == "out_on_r" else torch.empty_like(I0)
    est = r.view(B, 1) if which == "est_on_r" else V if which == "est_on_V" else torch.empty_like(e0)
    I = net.predict(G, V, r, out=out, est=est)
    assert torch.equal(I, I0) and torch.equal(est, e0)
    G2 = G.view(-1)[:B * n].view(B, n)
    with pytest.raises(_lib.XbarError):
        net.predict(G, V, r, out=G2)


def _both_paths(net, G, V, r):
    """(I, est) in one pass and layer by layer, and the layers' last map."""
    import torch

    from paper_2410_19993_amd import _lib
    B, m, n = G.shape
    e1, e2, I2 = (torch.empty((B, n), dtype=torch.float64, device="cuda") for _ in range(3))
    I1 = net.predict(G, V, r, est=e1)
    Y = net.forward(G, V, r)
    _lib.xbar_sg_predict(B, m, n, Y, G, V, I2, e2, net._stream())
    return [x.cpu().numpy() for x in (I1, e1, I2, e2, Y)]


@pytest.mark.parametrize("depth,C", [(2, 9), (3, 32), (4, 20), (5, 8)])
@pytest.mark.parametrize("B,m,n", [(3, 1, 70), (2, 8, 33), (2, 17, 100), (1, 40, 65)])
def test_one_pass_inference_has_the_bits_of_the_layers(B, m, n, depth, C):
    """The last map has the same bits.  A column's sum of m float32 values is exact in float64
    in any order while m max |Y| 2^24 < 2^53 min |Y|, which holds here, so the currents and
    estimates have the same bits too."""
    import torch

    from paper_2410_19993_amd.surrogate import Surrogate
    rng = np.random.default_rng(500 * depth + m + n)
    log(f"case infer bits B={B} {m}x{n} depth={depth} C={C}")
    G = torch.from_numpy(np.exp(rng.uniform(np.log(1e-6), np.log(1e-4), (B, m, n)))).cuda()
    V = torch.from_numpy(rng.uniform(0.0, 0.5, (B, m))).cuda()
    r = torch.from_numpy(rng.uniform(1.0, 5.0, B)).cuda()
    I1, e1, I2, e2, Y = _both_paths(Surrogate(channels=C, seed=4, depth=depth, zero_last=False), G, V, r)
    y = np.abs(Y.astype(np.float64))
    assert m * y.max() * 2.0 ** 24 < 2.0 ** 53 * y[y > 0].min()
    assert np.array_equal(I1, I2) and np.array_equal(e1, e2)


@pytest.mark.parametrize("what", ["nan", "zero", "inf", "overflow"])
@pytest.mark.parametrize("depth", [2, 4])
def test_one_pass_inference_of_values_that_are_not_finite(what, depth):
    """Conductances that are NaN, zero (log-conductance -inf) or infinite, and weights whose
    activations overflow: NaN and infinities come out where the layers give them, and other
    columns and samples are the layers' too."""
    import torch

    from paper_2410_19993_amd.surrogate import Surrogate
    rng = np.random.default_rng(60 + depth)
    log(f"case infer {what} depth={depth}")
    B, m, n = 3, 19, 70
    G = torch.from_numpy(np.exp(rng.uniform(np.log(1e-6), np.log(1e-4), (B, m, n)))).cuda()
    V = torch.from_numpy(rng.uniform(0.0, 0.5, (B, m))).cuda()
    r = torch.from_numpy(rng.uniform(1.0, 5.0, B)).cuda()
    net = Surrogate(channels=13, seed=4, depth=depth, zero_last=False)
    if what == "overflow":
        net.params *= 1e20
    else:
        G[1, 7, 40] = {"nan": float("nan"), "zero": 0.0, "inf": float("inf")}[what]
    I1, e1, I2, e2, Y = _both_paths(net, G, V, r)
    tol = 4 * m * np.finfo(float).eps
    for x, y in ((I1, I2), (e1, e2)):
        assert np.array_equal(np.isnan(x), np.isnan(y)) and np.array_equal(np.isinf(x), np.isinf(y))
        ok = np.isfinite(y)
        assert np.all(np.abs(x[ok] - y[ok]) <= 50 * tol * np.abs(y[ok]))
    assert what != "overflow" or not np.isfinite(Y).all()
