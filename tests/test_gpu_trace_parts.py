"""The shading path's shadow rays at the edges of the traversal's rules, hit
bits against brute force: launches whose tiles are shared by several
workgroups (one pixel, parts of one wavefront, ragged last tiles, one tile
fewer and more than fill the chip), meshes around the number of hoisted nodes,
and scenes with few and many big triangles."""

import numpy as np
import pytest

from workloads import make_workload
from tests.parity_util import to_np
from tests.test_gpu_wavefront_trace import _flags, _origins

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cu(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _check(verts, tris, env, n, spp, seed, reach=1.5):
    """n pixels with random positions within reach and random normals."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_03380_amd as M
    r = np.random.Generator(np.random.PCG64(seed))
    pos = r.uniform(-reach, reach, (3, n)).astype(np.float32)
    nrm = r.normal(size=(3, n)).astype(np.float32)
    scene, probe = M.Scene(_cu(verts), _cu(tris)), M.Env(_cu(env))
    korm = np.stack([np.ones(n), r.uniform(0.1, 1, n), r.uniform(0, 1, n)]).astype(np.float32)
    gb = M.GBuffer(_cu(pos), _cu(nrm), _cu(np.full((3, n), 0.5, np.float32)), _cu(korm), _cu(np.ones(n, np.uint8)),
                   _cu(np.array([[0.0, 0.0, 6.0]], np.float32)), 1, 1, n, 0)
    _, _, hb, dec = M.shade_fwd(scene, probe, gb, spp, seed=3, ray_eps=1e-3, decisions="dirs")
    d = to_np(dec).view(np.uint32)
    bits = to_np(hb).view(np.uint32)
    org = _origins(pos, nrm, 1e-3)
    lt, _, bt, _ = _flags()
    expect = np.zeros_like(bits)
    for t, flag in enumerate((lt, bt)):
        pix, smp = np.nonzero(d[..., 2] & flag)
        if len(pix) == 0:
            continue
        dirs = np.ascontiguousarray(d[pix, smp, 3 + 3 * t:6 + 3 * t]).view(np.float32)
        o, w = _cu(org[:, pix]), _cu(dirs.T)
        brute = to_np(M.trace_anyhit(scene, o, w, mode="brute")).astype(np.uint32)
        for mode in ("binary", "wide"):
            assert np.array_equal(to_np(M.trace_anyhit(scene, o, w, mode=mode)), brute), mode
        slot = 2 * smp + t
        np.bitwise_or.at(expect, (slot >> 5, pix), brute << (slot & 31).astype(np.uint32))
    assert np.array_equal(bits, expect)
    return scene.info()


@pytest.mark.parametrize("n,spp", [(1, 1), (1, 17), (63, 3), (257, 33), (4096, 4), (2047 * 256 + 1, 1),
                                   (2047 * 256, 1), (1024 * 256 - 1, 2)])
def test_split_tiles(n, spp):
    w = make_workload("tiny")
    _check(w.verts, w.tris, w.env, n, spp, n + spp)


def _soup(nt, size, seed):
    r = np.random.Generator(np.random.PCG64(seed))
    v = (r.uniform(-1, 1, (nt, 1, 3)) + size * r.normal(size=(nt, 3, 3))).astype(np.float32)
    return v.reshape(-1, 3), np.arange(3 * nt, dtype=np.int32).reshape(nt, 3)


@pytest.mark.parametrize("nt", [1, 2, 3, 4, 5, 9, 60, 90, 121, 257, 4000])
def test_mesh_sizes(nt):
    v, f = _soup(nt, 0.05, nt)
    _check(v, f, make_workload("tiny").env, 3000, 3, nt)


@pytest.mark.parametrize("n_big", [1, 2, 3, 36, 127, 128, 129, 200])
def test_big_triangles(n_big):
    v, f = _soup(500, 0.02, n_big)
    bv, bf = _soup(n_big, 0.8, n_big + 1)
    info = _check(np.concatenate([v, bv]), np.concatenate([f, bf + len(v)]), make_workload("tiny").env, 3000, 3, n_big)
    assert info["n_big"] >= n_big * 0.8
