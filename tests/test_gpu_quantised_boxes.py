"""The half-precision node boxes are conservative: the binary and the 4-wide
walk answer like brute force on scenes whose frames are hard to quantise."""

import numpy as np
import pytest

from tests.parity_util import to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SCENES = {
    "unit": (1.0, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0)),
    "far": (1.0, (3e4, -2e4, 1e4), (1.0, 1.0, 1.0)),           # a small scene far from the origin
    "tiny": (1e-5, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0)),
    "huge": (1e12, (1e11, 0.0, 0.0), (1.0, 1.0, 1.0)),
    "flat": (1.0, (0.0, 0.25, 0.0), (1.0, 0.0, 1.0)),          # no extent along y
    "needle": (1.0, (0.0, 0.0, 0.0), (1.0, 1e-6, 1e-6)),
}


@pytest.mark.parametrize("name", sorted(SCENES))
def test_walks_equal_brute_force(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_03380_amd as M
    scale, offset, squash = SCENES[name]
    r = np.random.Generator(np.random.PCG64(len(name)))
    nt, n = 3000, 20000
    squash, offset = np.array(squash), np.array(offset)
    centre = r.uniform(-1, 1, (nt, 1, 3))
    size = 10.0 ** r.uniform(-4, -0.7, (nt, 1, 1))
    v = ((centre + size * r.normal(size=(nt, 3, 3))) * squash * scale + offset).astype(np.float32)
    f = np.arange(3 * nt, dtype=np.int32).reshape(nt, 3)
    # rays at points of the triangles, from points among them and beside them
    w = r.dirichlet((1, 1, 1), n)
    target = np.einsum("nk,nkc->nc", w, v[r.integers(0, nt, n)].astype(np.float64))
    o = (r.uniform(-1.2, 1.2, (n, 3)) * np.maximum(squash, 0.3) * scale + offset).astype(np.float32)
    d = target - o
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    cu = lambda x: torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()  # noqa: E731
    scene = M.Scene(cu(v.reshape(-1, 3)), torch.from_numpy(f).cuda())
    ot, dt = cu(o.T), cu(d.T)
    brute = to_np(M.trace_anyhit(scene, ot, dt, mode="brute"))
    assert 0 < brute.sum()
    for mode in ("binary", "wide"):
        assert np.array_equal(to_np(M.trace_anyhit(scene, ot, dt, mode=mode)), brute), mode
