"""The probe gradient's fixed-point sums where a small image meets a large probe:
many buckets, few records, and those in two neighbouring buckets.  A sum takes at
most 2^10 records there, so one record is rounded by at most 2^-53 of the power
of two above its bucket's largest value.  Gradients 2^-40 of the bucket's largest
keep that many bits beside it."""

import numpy as np
import pytest

from workloads import make_workload
from tests.parity_util import to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_small_gradients_beside_large():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_03380_amd as M
    w = make_workload("tiny")
    spp, H, W, row = 16, 1024, 2048, 256
    env = np.zeros((H, W, 3), np.float32)
    env[row] = 1.0                              # 2048 texels of equal probability: none is summed apart
    cu = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    scene, probe, gb = M.Scene(cu(w.verts), cu(w.tris)), M.Env(cu(env)), M.GBuffer.from_workload(w, "cuda")
    _, _, hb, dec = M.shade_fwd(scene, probe, gb, spp, seed=3, ray_eps=w.ray_eps, decisions=True)

    def grad(u):
        g = cu(np.broadcast_to(u, (3, gb.n)).astype(np.float32))
        return to_np(M.shade_bwd(scene, probe, gb, spp, g, g, hitbits=hb, seed=3, ray_eps=w.ray_eps)[3]).reshape(-1, 3)

    large = np.zeros(gb.n)
    large[np.nonzero(w.mask.reshape(-1))[0][100::700]] = 1.0
    r = np.random.default_rng(4)
    small = r.uniform(0.5, 1.0, gb.n) * 2.0 ** -40 * (large == 0)
    both, alone, big = (grad(u).astype(np.float64) for u in (large + small, small, large))
    # samples of a texel, and the largest gradient of its bucket of 1024
    d = to_np(dec).view(np.uint32)
    n = sum(np.bincount(t[t < H * W].astype(np.int64), minlength=H * W) for t in (d[..., 0], d[..., 1]))
    top = np.repeat(big.reshape(-1, 1024 * 3).max(1), 1024)[:, None]
    t = np.arange(row * W, (row + 1) * W)
    keep = t[(big[t] == 0).all(1) & (alone[t] > 0).all(1) & (top[t, 0] > 0)]
    assert len(keep) > 500
    tol = n[keep, None] * 2.0 ** -53 * 2.0 * top[keep] + 16 * 2.0 ** -24 * alone[keep]
    err = np.abs(both - alone)[keep]
    assert (err <= tol).all(), "worst %.3g of the bound" % (err / tol).max()
