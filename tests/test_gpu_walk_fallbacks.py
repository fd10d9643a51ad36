"""Walks of the 4-wide hierarchy whose stacks overflow, which hand the ray to the
binary nodes: a query lane's (14 entries in LDS, 32 in private memory), and a
wavefront's shared one (1152 entries in queries, 1024 in the edge gradient).
The meshes are slivers without area whose boxes all hold the middle of the
scene, so a ray through it hits every box, and whose centroids make deep
subtrees; the walks' stacks are replayed here over the built tree.  What a ray
can hit lies where its walk comes last."""

import numpy as np
import pytest

import oracle
from tests.parity_util import to_np
from workloads import make_workload
from workloads.configs import from_arrays

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cu(x, t=np.float32):
    return torch.from_numpy(np.ascontiguousarray(x, t)).cuda()


def _slivers(c):
    d = np.array([0.75, 0.75, 0.75])
    return np.stack([c - d, c + d, c], 1)


def _triangle(at, size):
    """A triangle around `at`, across the direction (1, 1, 1)."""
    return at + size * np.array([[1.0, -1.0, 0.0], [0.0, 1.0, -1.0], [-1.0, 0.0, 1.0]])


def _scene(tri):
    import paper_2206_03380_amd as M
    v = np.concatenate(tri).astype(np.float32).reshape(-1, 3)
    f = np.arange(len(v), dtype=np.int32).reshape(-1, 3)
    return M.Scene(_cu(v), _cu(f, np.int32)), v, f


def _children(esc, pay, x):
    """Slots of the wide node at binary node x: None (unused) or (node, is a leaf)."""
    out = [None] * 4
    for i, y in enumerate((x + 1, esc[x + 1])):
        if pay[y] != 0:
            out[2 * i] = (y, True)
        else:
            out[2 * i], out[2 * i + 1] = (((z, pay[z] != 0)) for z in (y + 1, esc[y + 1]))
    return out


def _lane_peak(esc, pay):
    """Most entries of a lane that takes each split's first child first."""
    stack, peak = [0], 0
    while stack:
        x = stack.pop()
        if pay[x] == 0:
            stack += [s[0] for s in _children(esc, pay, x)[::-1] if s]
            peak = max(peak, len(stack))
    return peak


def _wave_overflows(esc, pay, cap):
    """Leaves that a wavefront's walk with every box hit has tested when its stack
    overflows, None if it never does."""
    stack, tested = [(0, False)], set()
    while stack:
        take = min(len(stack), 64, max((cap - len(stack)) // 3, 1))
        top, stack = stack[-take:], stack[:-take]
        tested |= {x for x, leaf in top if leaf}
        kids = [_children(esc, pay, x) for x, leaf in top if not leaf]
        stack += [k[s] for s in range(4) for k in kids if k[s]]
        if len(stack) > cap:
            return tested
    return None


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n", [1, 70, 3000])
def test_lane_stack(n):
    _need_gpu()
    import paper_2206_03380_amd as M
    # centroids at 0.6 of every power of two on the axes: each split of the keys takes one off
    c = np.concatenate([0.6 * 2.0 ** -k * np.eye(3) for k in range(21)] + [np.eye(3), np.zeros((1, 3))])
    sc, _, _ = _scene([_slivers(c), _triangle(np.full(3, 0.9), 0.15)[None]])
    nodes = to_np(sc.nodes()[0])
    assert _lane_peak(nodes[:, 3], nodes[:, 7]) > 14 + 32 + 4
    r = np.random.default_rng(n)
    o = 2.0 + r.uniform(-0.3, 0.3, (n, 3))
    d = r.uniform(0.4, 0.6, (n, 3)) - o
    o, d = _cu(o.T), _cu(d.T)
    hit = M.trace_anyhit(sc, o, d)
    brute = M.trace_anyhit(sc, o, d, mode="brute")
    assert torch.equal(hit, brute)
    if n > 1:
        assert 0.1 * n < int(brute.sum()) < 0.9 * n


def _bushy():
    """Centroids by their keys: 64 cells (six bits), in each a chain whose every
    level (two bits) has three leaves of two triangles before the next level."""
    keys = []
    for cell in range(64):
        for level in range(10):
            keys += [(cell, "11" * level + s) for s in ("00", "01", "10")]
    c = np.zeros((len(keys), 3))
    for i, (cell, path) in enumerate(keys):
        bits = format(cell, "06b") + path + "1"          # (inside its interval)
        for k, b in enumerate(bits):
            c[i, k % 3] += int(b) * 2.0 ** -(k // 3 + 1)
    return np.repeat(c, 2, 0)


def test_wave_stack_of_queries():
    _need_gpu()
    import paper_2206_03380_amd as M
    sc, _, _ = _scene([_slivers(np.concatenate([_bushy(), np.ones((1, 3))])), _triangle(np.zeros(3), 0.1)[None]])
    nodes = to_np(sc.nodes()[0])
    tested = _wave_overflows(nodes[:, 3], nodes[:, 7], 18 * 64)
    first = int(np.nonzero(nodes[:, 7] != 0)[0][0])      # the leaf at the lowest key, which the rays can hit
    assert tested is not None and first not in tested
    r = np.random.default_rng(3)
    for n in (1, 2, 4):
        o = np.where(np.arange(n)[:, None] % 2 == 0, -1.0, [-1.0, -0.3, -0.3]) + r.uniform(-0.01, 0.01, (n, 3))
        d = r.uniform(0.49, 0.51, (n, 3)) - o
        o, d = _cu(o.T), _cu(d.T)
        hit = to_np(M.trace_anyhit(sc, o, d))
        assert np.array_equal(hit, to_np(M.trace_anyhit(sc, o, d, mode="brute")))
        assert np.array_equal(hit, (np.arange(n) % 2 == 0).astype(np.uint8))


def test_wave_stack_of_the_edge_gradient():
    _need_gpu()
    import paper_2206_03380_amd as M
    r = np.random.Generator(np.random.PCG64(5))
    # triangles around the middle, with silhouettes for the pixels in it and some behind others
    at = r.normal(size=(40, 3))
    at = 0.5 + at / np.linalg.norm(at, axis=1, keepdims=True) * r.uniform(0.5, 0.9, (40, 1))
    off = 0.25 * r.normal(size=(40, 3, 3))
    shell = np.clip(at, 0.01, 0.99)[:, None] + off - off.mean(1, keepdims=True)   # (centroids inside the cells)
    sc, v, f = _scene([_slivers(np.concatenate([_bushy(), np.zeros((1, 3)), np.ones((1, 3))])), shell])
    nodes = to_np(sc.nodes()[0])
    assert _wave_overflows(nodes[:, 3], nodes[:, 7], 1024) is not None
    n, n_es = 128, 64
    env = make_workload("tiny").env
    korm = np.stack([np.ones(n), r.uniform(0.3, 1, n), r.uniform(0, 1, n)], 1)
    w = from_arrays("shell", v, f, env, r.uniform(0.4, 0.6, (n, 3)), r.normal(size=(n, 3)), r.uniform(0, 1, (n, 3)),
                    korm, eye=[[0.0, 0.0, 7.0]], ray_eps=1e-4)
    verts, tris = _cu(w.verts), _cu(w.tris, np.int32)
    scene, probe, edges = M.Scene(verts, tris), M.Env(_cu(w.env)), M.Edges(tris, len(w.verts))
    gb = M.GBuffer.from_workload(w, "cuda")
    ud, us = r.normal(size=(3, n)).astype(np.float32), r.normal(size=(3, n)).astype(np.float32)
    st = M.new_stats()
    g = to_np(M.shade_bwd_edges(scene, probe, edges, verts, gb, n_es, _cu(ud), _cu(us), seed=4, ray_eps=w.ray_eps,
                                stats=st)).astype(np.float64)
    w.seed = 4
    o = oracle.edge_grad(w, oracle.mesh_edges(w.tris, len(w.verts)), n_es, ud.astype(np.float64), us.astype(np.float64))
    bound = 1e-4 * o["abs"] + 4.0 * o["cond"] + o["flag"] + 1e-7 * np.abs(o["g_verts"]).max()
    assert (np.abs(g - o["g_verts"]) <= np.maximum(bound, 1e-300)).all()
    assert o["traced"] >= 20 and o["blocked"] < o["traced"]
    assert abs(M.read_stats(st)["rays_traced"] - o["traced"]) <= o["flagged"]
