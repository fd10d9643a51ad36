"""The denoiser where the two components of a steep depth gradient cancel: in
each view the depth is G (3 x - y) but for the pixels with 3 x = y, whose depths
are a few times the prediction's epsilon apart.  Along that line the predicted
change is exactly zero, so the weights there are exp(-|dz| / eps) whatever G is;
a prediction of which one component was rounded before the sum is off by up to
2^-53 G.  Border pixels (one-sided differences of the small depths are not
exact) neither count nor send gradients.  Bounds as in the denoiser's parity
tests."""

import numpy as np
import pytest

from oracle import bilateral as B
from tests.test_bilateral import TOL, _footprint_max, _gpu_filter

pytestmark = pytest.mark.gpu


def _case(k, nc, sigma):
    """Twelve views with slopes of 13-bit significands times 2^k."""
    V, H, W = 12, 60, 30
    R = B.radius(sigma)
    rng = np.random.default_rng(13)
    G = (rng.integers(2 ** 12, 2 ** 13, V) * 2 + 1)[:, None, None] * 2.0 ** (k - 13)
    y, x = np.mgrid[0:H, 0:W]
    line = np.broadcast_to(3 * x == y, (V, H, W))
    z = (G * (3 * x - y)).astype(np.float32)
    assert np.array_equal(z.astype(np.float64), G * (3.0 * x - y))
    z[line] = (rng.integers(0, 4, line.sum()) * 1e-5).astype(np.float32)
    inner = (y > R) & (y < H - 1 - R) & (x > R) & (x < W - 1 - R)
    inner = np.broadcast_to(inner, (V, H, W)).reshape(-1)
    assert (inner & line.reshape(-1)).sum() > 5 * V
    n = V * H * W
    nrm = np.tile(np.array([[0.0], [0.0], [1.0]], np.float32), (1, n))
    c = rng.random((nc, n)).astype(np.float32)
    g = (rng.normal(size=(nc, n)) * inner).astype(np.float32)
    return V, H, W, R, z.reshape(-1), nrm, np.ones(n, np.uint8), c, g, inner


@pytest.mark.parametrize("k", [14, 27, 40, 42])
@pytest.mark.parametrize("nc,sigma,sigma_z", [(1, 1.3, 1.0), (3, 1.3, 0.7), (6, 2.0, 1.0), (3, 2.6, 0.3)])
def test_cancelling_gradients(k, nc, sigma, sigma_z):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sigma, sigma_z = float(np.float32(sigma)), float(np.float32(sigma_z))
    V, H, W, R, depth, nrm, mask, c, g, inner = _case(k, nc, sigma)
    out, wsum, gin = _gpu_filter(depth, nrm, mask, V, H, W, c, sigma, g, sigma_z)
    o_out, o_w = B.bilateral_fwd(c, depth, nrm, mask, V, H, W, sigma, sigma_z)
    bound = TOL * _footprint_max(c, mask, V, H, W, R) + 1e-7
    err = np.abs(out - o_out).max(0)
    assert np.all(err[inner] <= bound[inner]), "fwd: worst %.3g of bound" % (err / bound)[inner].max()
    assert np.all(np.abs(wsum - o_w)[inner] <= TOL * o_w[inner])
    o_g = B.bilateral_bwd(g, depth, nrm, mask, V, H, W, sigma, sigma_z)
    scale = B.bilateral_bwd(np.abs(g), depth, nrm, mask, V, H, W, sigma, sigma_z)
    gbound = TOL * scale + 1e-7 * np.abs(o_g).max()
    assert np.all(np.abs(gin - o_g) <= gbound), "bwd: worst %.3g of bound" % (np.abs(gin - o_g) / gbound).max()
