"""Light draws against a search of the whole tables (NumPy): probe shapes at the
edges of the padded marginal search, the guide cells and the 16-entry window
(rows of the window reach the next row and the table's end)."""

import numpy as np
import pytest

import oracle
from tests.parity_util import gpu_forward, to_np
from workloads import make_workload

torch = pytest.importorskip("torch")


def test_reciprocal_division():
    """The quotient by an image side from its reciprocal (one correction by the
    exact remainder) is the rounded quotient, here over every significand."""
    a = np.arange(1 << 23, 1 << 24, dtype=np.float32) * np.float32(2.0 ** -23)
    for b in (1, 3, 7, 203, 389, 1023, 1025, 2047, 3333, 4093, 4095):
        rb = np.float32(1) / np.float32(b)
        q = a * rb
        # FP64 stands for the fused operations: the remainder is exact in it,
        # and the sum has 48 + 24 bits, rounded to 53 and then to 24
        e = (a.astype(np.float64) - q.astype(np.float64) * b).astype(np.float32)
        got = (q.astype(np.float64) + e.astype(np.float64) * np.float64(rb)).astype(np.float32)
        assert np.array_equal(got, a / np.float32(b)), b


@pytest.mark.gpu
@pytest.mark.parametrize("H,W", [(1, 1), (1, 15), (2, 16), (3, 17), (5, 4096), (33, 2047), (63, 31), (64, 64),
                                 (65, 129), (1025, 1023), (600, 2048)])
def test_light_draws(H, W):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = make_workload("tiny")
    r = np.random.Generator(np.random.PCG64(H * 5000 + W))
    e = r.lognormal(0, 2.5, (H, W, 3)).astype(np.float32)
    e[r.random((H, W)) < 0.3] = 0.0
    e[H - 1, W - 1] = 50.0                      # the last row's last columns are drawn
    e[H // 2, :] = 1.0                          # one column per CDF step
    w.env = e
    out, (_, env, _, _) = gpu_forward(w, spp=64, seed=9)
    cond, marg = (to_np(t) for t in env.tables()[:2])
    dec = out["decisions"][..., 0]
    n, spp = dec.shape
    hw = w.height * w.width
    pix = np.repeat(np.arange(n), spp)
    s = np.tile(np.arange(spp), n)
    xi = oracle.uniforms(9, pix % hw, w.view_base + pix // hw, s).astype(np.float32)
    i = np.minimum(np.searchsorted(marg, xi[:, 0], side="right") - 1, H - 1)
    j = np.empty_like(i)
    for k in np.unique(i):
        m = i == k
        j[m] = np.minimum(np.searchsorted(cond[k], xi[m, 1], side="right") - 1, W - 1)
    ref = (i * W + j).astype(np.uint32)
    got = dec.reshape(-1)
    drawn = got != 0xFFFFFFFF
    assert drawn.mean() > 0.05
    assert np.array_equal(got[drawn], ref[drawn])
