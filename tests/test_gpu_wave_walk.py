"""The edge gradient's out-side rays walked by whole wavefronts, on scenes at
the edges of that walk (one node, a few, a stack that overflows) against the
oracle's traced and blocked counts and its gradient's bound."""

import numpy as np
import pytest

import oracle
from workloads import make_workload
from workloads.configs import from_arrays
from tests.parity_util import to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt,spread", [(1, 0.5), (2, 0.5), (5, 0.5), (300, 0.2), (6000, 2.0)])
def test_wave_walk(nt, spread):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_03380_amd as M
    r = np.random.Generator(np.random.PCG64(nt))
    v = (r.uniform(-1, 1, (nt, 1, 3)) + spread * r.normal(size=(nt, 3, 3))).reshape(-1, 3)
    f = np.arange(3 * nt).reshape(nt, 3)
    n = 64
    env = make_workload("tiny").env
    korm = np.stack([np.ones(n), r.uniform(0.3, 1, n), r.uniform(0, 1, n)], 1)
    w = from_arrays("soup", v, f, env, r.uniform(-1.2, 1.2, (n, 3)), r.normal(size=(n, 3)), r.uniform(0, 1, (n, 3)),
                    korm, eye=[[0.0, 0.0, 7.0]], ray_eps=1e-3)
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    verts, tris = cu(w.verts), cu(w.tris)
    scene, probe, edges = M.Scene(verts, tris), M.Env(cu(w.env)), M.Edges(tris, len(w.verts))
    gb = M.GBuffer.from_workload(w, "cuda")
    ud, us = r.normal(size=(3, n)).astype(np.float32), r.normal(size=(3, n)).astype(np.float32)
    st = M.new_stats()
    n_es = 16
    g = to_np(M.shade_bwd_edges(scene, probe, edges, verts, gb, n_es, cu(ud), cu(us), seed=4, ray_eps=w.ray_eps,
                                stats=st)).astype(np.float64)
    w.seed = 4
    o = oracle.edge_grad(w, oracle.mesh_edges(w.tris, len(w.verts)), n_es, ud.astype(np.float64), us.astype(np.float64))
    bound = 1e-4 * o["abs"] + 4.0 * o["cond"] + o["flag"] + 1e-7 * np.abs(o["g_verts"]).max()
    assert (np.abs(g - o["g_verts"]) <= np.maximum(bound, 1e-300)).all()
    assert abs(M.read_stats(st)["rays_traced"] - o["traced"]) <= o["flagged"]
