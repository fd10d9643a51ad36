"""Rays through a triangle's edges are decided by the last bit of the sheared
coordinates: every traversal gives the rounding that the test defines (one or
two roundings by the ray's axis), here computed on the CPU.  The directions'
largest component is a power of two, so its reciprocal is exact; the FP64 sums
stand for fused ones (a second rounding changes one in 2^29)."""

import numpy as np
import pytest

from tests.parity_util import to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
F, D = np.float32, np.float64


def _hits(tri, o, d, kz, fused):
    """fused: {kz: (row kx, row ky)} of the cyclic axes after kz."""
    n = len(o)
    i = np.arange(n)
    kx, ky = (kz + 1) % 3, (kz + 2) % 3
    rz = F(1) / d[i, kz]
    row = []
    for k, which in ((kx, 0), (ky, 1)):
        s = d[i, k] * rz
        f = np.array([fused[a][which] for a in range(3)])[kz]
        out = []
        for v in tri:
            z, x = v[kz] - o[i, kz], v[k] - o[i, k]
            out.append(np.where(f, (D(1) * x - D(1) * s * z).astype(F), x - s * z))
        row.append(out)
    (ax, bx, cx), (ay, by, cy) = row
    e = [cx * by - cy * bx, ax * cy - ay * cx, bx * ay - by * ax]
    zero = (e[0] == 0) | (e[1] == 0) | (e[2] == 0)
    w = lambda x: x.astype(D)  # noqa: E731
    e64 = [(w(cx) * w(by) - w(cy) * w(bx)), (w(ax) * w(cy) - w(ay) * w(cx)), (w(bx) * w(ay) - w(by) * w(ax))]
    u, v, q = (np.where(zero, b.astype(F), a) for a, b in zip(e, e64))
    mixed = ((u < 0) | (v < 0) | (q < 0)) & ((u > 0) | (v > 0) | (q > 0))
    det = u + v + q
    z = [rz * (p[kz] - o[i, kz]) for p in tri]
    t = u * z[0] + v * z[1] + q * z[2]
    return ~mixed & (det != 0) & np.where(det > 0, t > 0, t < 0)


def test_shear_rounding():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_03380_amd as M
    r = np.random.Generator(np.random.PCG64(41))
    n = 300000
    # a second, far triangle gives the hierarchy two leaves
    tri = r.uniform(-1, 1, (3, 3)).astype(F)
    v = np.concatenate([tri, tri + F(1000)])
    a, b = tri[r.integers(0, 3, n)], tri[r.integers(0, 3, n)]
    w = r.uniform(0, 1, (n, 1))
    p = a * w + b * (1 - w)
    kz = r.integers(0, 3, n)
    d = r.uniform(-1, 1, (n, 3)).astype(F)
    d[np.arange(n), kz] = r.choice((-1, 1), n)
    o = (p - d * r.uniform(0.5, 2, (n, 1))).astype(F)
    fused = {0: (True, False), 1: (False, False), 2: (True, True)}
    ref = _hits(tri, o, d, kz, fused)
    assert 0.2 < ref.mean() < 0.8
    # the inputs tell the roundings apart
    for other in ({k: (True, True) for k in range(3)}, {k: (False, False) for k in range(3)}):
        assert (_hits(tri, o, d, kz, other) != ref).sum() > 100
    sc = M.Scene(torch.from_numpy(v).cuda(), torch.arange(6, dtype=torch.int32, device="cuda").reshape(2, 3))
    od, dd = (torch.from_numpy(np.ascontiguousarray(x.T)).cuda() for x in (o, d))
    for mode in ("brute", "binary", "wide"):
        got = to_np(M.trace_anyhit(sc, od, dd, mode=mode)).astype(bool)
        assert np.array_equal(got, ref), (mode, int((got != ref).sum()))
