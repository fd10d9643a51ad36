"""The quotients of light samples' coordinates by the probe's sides are the rounded
ones, on the device: directions near the horizon and near the planes where a
component passes through zero, against FP64 sines and cosines of the quotients
that NumPy rounds.  There a component is small and exact to 2 ulp (4 u, u = 2^-24)
for each sine or cosine in it and one rounding (2 u) for their product, while a
quotient one ulp off moves it by at least pi u / 2."""

import numpy as np
import pytest

import oracle
from tests.parity_util import gpu_forward, to_np
from workloads import make_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
F, D, U = np.float32, np.float64, 2.0 ** -24


@pytest.mark.parametrize("H,W", [(3, 7), (17, 31), (63, 129), (203, 389), (600, 1025), (1025, 2047), (64, 128)])
def test_quotients(H, W):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = make_workload("tiny")
    r = np.random.Generator(np.random.PCG64(H * 5000 + W))
    w.env = r.lognormal(0, 0.5, (H, W, 3)).astype(F)
    out, (_, env, _, _) = gpu_forward(w, spp=64, seed=9)
    cond, marg = (to_np(t) for t in env.tables()[:2])
    dec = out["decisions"][..., 0]
    n, spp = dec.shape
    hw = w.height * w.width
    pix, s = np.repeat(np.arange(n), spp), np.tile(np.arange(spp), n)
    xi = oracle.uniforms(9, pix % hw, w.view_base + pix // hw, s).astype(F)
    t = dec.reshape(-1)
    k = np.nonzero(t != 0xFFFFFFFF)[0]
    i, j = (t[k] // W).astype(np.int64), (t[k] % W).astype(np.int64)
    x0, x1 = xi[k, 0], xi[k, 1]
    m0, m1, c0, c1 = marg[i], marg[i + 1], cond[i, j], cond[i, j + 1]
    v = (i.astype(F) + (x0 - m0) / (m1 - m0)) / F(H)
    u = (j.astype(F) + (x1 - c0) / (c1 - c0)) / F(W)
    assert v.dtype == F and u.dtype == F
    got = out["dirs"][..., 0, :].reshape(-1, 3)[k].astype(D)
    # cos and sin of pi x near their zeros, by the exact distance to them
    ct, st = np.sin(np.pi * (0.5 - v.astype(D))), np.sin(np.pi * v.astype(D))
    u2 = 2.0 * u.astype(D)
    sp = np.sin(np.pi * (u2 - np.round(u2))) * (-1.0) ** np.round(u2)
    near = np.abs(ct) < 0.05
    assert near.sum() > 200
    assert (np.abs(got[:, 1] - ct)[near] <= 4 * U * np.abs(ct[near])).all()
    near = (np.abs(sp) < 0.05) & (st > 0.5)
    assert near.sum() > 200
    assert (np.abs(got[:, 2] - st * sp)[near] <= 10 * U * np.abs(st * sp)[near]).all()
    # and a quotient one ulp off is told apart
    off = np.sin(np.pi * (0.5 - np.nextafter(v, F(1)).astype(D)))
    near = (np.abs(ct) < 0.05) & (ct != 0)
    assert (np.abs(off - ct)[near] > 4 * U * np.abs(ct[near])).all()
