"""Shadow rays of launches whose tiles are shared by several workgroups, at the
edges of the split: one pixel, parts of one wavefront, ragged last tiles, and
one tile fewer and more than fill the chip.  Hit bits equal brute force."""

import numpy as np
import pytest

from workloads import make_workload
from tests.parity_util import to_np
from tests.test_gpu_wavefront_trace import _flags, _origins

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,spp", [(1, 1), (1, 17), (63, 3), (257, 33), (4096, 4), (2047 * 256 + 1, 1),
                                   (2047 * 256, 1), (1024 * 256 - 1, 2)])
def test_split_tiles_equal_brute_force(n, spp):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_03380_amd as M
    w = make_workload("tiny")
    r = np.random.Generator(np.random.PCG64(n + spp))
    pos = r.uniform(-1.5, 1.5, (3, n)).astype(np.float32)
    nrm = r.normal(size=(3, n)).astype(np.float32)
    cu = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    scene, env = M.Scene(cu(w.verts), cu(w.tris)), M.Env(cu(w.env))
    korm = np.stack([np.ones(n), r.uniform(0.1, 1, n), r.uniform(0, 1, n)]).astype(np.float32)
    gb = M.GBuffer(cu(pos), cu(nrm), cu(np.full((3, n), 0.5, np.float32)), cu(korm), cu(np.ones(n, np.uint8)),
                   cu(np.array([[0.0, 0.0, 6.0]], np.float32)), 1, 1, n, 0)
    _, _, hb, dec = M.shade_fwd(scene, env, gb, spp, seed=3, ray_eps=1e-3, decisions="dirs")
    d = to_np(dec).view(np.uint32)
    bits = to_np(hb).view(np.uint32)
    org = _origins(pos, nrm, 1e-3)
    lt, _, bt, _ = _flags()
    traced = 0
    for t, flag in enumerate((lt, bt)):
        pix, smp = np.nonzero(d[..., 2] & flag)
        dirs = np.ascontiguousarray(d[pix, smp, 3 + 3 * t:6 + 3 * t]).view(np.float32)
        traced += len(pix)
        if len(pix) == 0:
            continue
        brute = to_np(M.trace_anyhit(scene, cu(org[:, pix]), cu(dirs.T), brute=True)).astype(bool)
        slot = 2 * smp + t
        assert np.array_equal((bits[slot >> 5, pix] >> (slot & 31)) & 1, brute)
    # no bit of a sample that was not traced
    assert traced >= int(sum(bin(int(x)).count("1") for x in bits.reshape(-1)[:100000]))
