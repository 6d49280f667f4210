"""The learned index's gradient where a parameter or a target is infinite or NaN:
an input bit chooses which weights are added, so a bit that is not set keeps its
weights out of a sample, and its gradients free of that sample, whatever they hold."""
import numpy as np
import pytest

import synth
from tests._util import dev_u32, say
from tests.test_zz_no_alloc import _bf16, _params, _split

pytestmark = pytest.mark.gpu
mbr = pytest.importorskip("paper_2203_04158_amd")
torch = pytest.importorskip("torch")


def _want(p32, q, tgt):
    """Loss and gradients in fp64, sums over the set bits only."""
    W1, b1, W2, b2, w3, b3 = [np.asarray(a, dtype=np.float64) for a in _split(_bf16(p32))]
    X = ((q[:, None] >> np.arange(32, dtype=np.uint64)) & np.uint64(1)) == 1
    with np.errstate(all="ignore"):
        z1 = b1 + np.where(X[:, None, :], W1[None], 0.0).sum(-1)
        h1 = np.where(z1 > 0, z1, 0.0)
        z2 = b2 + (h1[:, None, :] * W2[None]).sum(-1)
        h2 = np.where(z2 > 0, z2, 0.0)
        y = b3 + (h2 * w3).sum(-1)
        dy = 2 * (y - tgt) / len(q)
        dz2 = (z2 > 0) * dy[:, None] * w3
        dz1 = np.where(h1 > 0, (dz2[:, :, None] * W2[None]).sum(1), 0.0)
        g = [np.where(X[:, None, :], dz1[:, :, None], 0.0).sum(0), dz1.sum(0), (dz2[:, :, None] * h1[:, None, :]).sum(0), dz2.sum(0),
             (dy[:, None] * h2).sum(0), dy.sum()]
        return np.mean((y - tgt) ** 2), g


def _check(p32, q, tgt):
    g, loss = mbr.mlp_gradients(torch.from_numpy(p32).cuda(), dev_u32(q), torch.from_numpy(tgt).cuda())
    want_loss, want = _want(p32, q, tgt.astype(np.float64))
    assert np.isclose(float(loss.cpu()[0]), want_loss, rtol=1e-5, equal_nan=True)
    for a, b in zip(_split(g.cpu().numpy()), want):
        a, b = np.atleast_1d(a).ravel(), np.atleast_1d(b).ravel()
        assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(a[np.isinf(a)], b[np.isinf(b)])
        ok = np.isfinite(b)
        if ok.any():  # the gradient test's bar
            assert np.abs(a[ok] - b[ok]).max() <= 1e-4 * max(1e-12, np.abs(b[ok]).max())
    return want


@pytest.mark.parametrize("B", [64, 8256])
@pytest.mark.parametrize("v", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("set_in", ["none", "one"])
def test_non_finite_weight_of_a_bit(B, v, set_in):
    say("gradient, non-finite first-layer weight", v, "batch", B, "bit set in", set_in)
    p = _params(31).copy()
    p[7 * 32 + 20] = v  # unit 7, bit 20
    q = synth.splitmix64(40, B) & np.uint64(0xFFEFFFFF)
    tgt = synth.uniform01(41, B).astype(np.float32)
    if set_in == "one":
        q[B - 3] |= np.uint64(1 << 20)
    want = _check(p, q, tgt)
    if set_in == "none":
        assert all(np.isfinite(a).all() for a in want)


@pytest.mark.parametrize("v", [np.inf, np.nan])
def test_non_finite_target(v):
    p = _params(33)
    q = synth.splitmix64(42, 128) & np.uint64(0x00FFFFFF)
    tgt = synth.uniform01(43, 128).astype(np.float32)
    tgt[70] = v
    want = _check(p, q, tgt)
    assert np.isfinite(want[0][:, 24:]).all() and not np.isfinite(want[0]).all()  # the top bits are set in no sample
