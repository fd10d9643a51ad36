"""Any-hit queries over the 4-wide hierarchy against every triangle: ray counts
at the edges of waves, workgroups and their chunks, scenes that fill a lane's
stack and leave a few long rays to the whole wave, and rays that are not
finite."""

import numpy as np
import pytest

from tests.parity_util import to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _mesh(kind, r):
    if kind == "soup":                      # overlapping triangles: many pending boxes
        v = (r.uniform(-0.2, 0.2, (3000, 1, 3)) + 0.5 * r.normal(size=(3000, 3, 3))).astype(np.float32)
    elif kind == "sheets":                  # slivers along the rays: long walks
        k = 4000
        a = r.uniform(-1, 1, (k, 1, 3)) * [1, 0.01, 1]
        v = (a + r.uniform(-1, 1, (k, 3, 3)) * [0.002, 0.0001, 0.5]).astype(np.float32)
    else:                                   # a fine grid
        g = np.stack(np.meshgrid(np.linspace(-1, 1, 60), np.linspace(-1, 1, 60), indexing="ij"), -1)
        p = np.concatenate([g, 0.1 * np.sin(3 * g[..., :1])], -1)
        q = np.stack([p[:-1, :-1], p[1:, :-1], p[1:, 1:], p[:-1, :-1], p[1:, 1:], p[:-1, 1:]], 2)
        v = q.reshape(-1, 3, 3).astype(np.float32)
    return v.reshape(-1, 3), np.arange(3 * len(v), dtype=np.int32).reshape(-1, 3)


@pytest.mark.parametrize("kind,n", [("grid", 1), ("grid", 63), ("grid", 65), ("sheets", 257), ("soup", 1000),
                                    ("sheets", 20001), ("grid", 2048 * 256 - 1), ("grid", 2048 * 256 + 1),
                                    ("soup", 600001), ("grid", 2048 * 4096 + 5)])
def test_queries(kind, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_03380_amd as M
    r = np.random.Generator(np.random.PCG64(n))
    v, f = _mesh(kind, r)
    sc = M.Scene(torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda())
    gen = torch.Generator(device="cuda").manual_seed(n)
    o = torch.randn((3, n), generator=gen, device="cuda")
    d = torch.randn((3, n), generator=gen, device="cuda")
    if kind != "soup":                      # towards the surface, and along it
        o = 1.5 * o / o.norm(dim=0)
        d = 0.8 * torch.rand((3, n), generator=gen, device="cuda") - 0.4 - o
    if n > 1000:
        d[:, ::97] = float("nan")
        d[1, ::89] = 0.0
        d[:, ::83] = 0.0
        o[0, ::79] = float("inf")
    hit = M.trace_anyhit(sc, o, d)
    assert hit.shape == (n,) and int(hit.max()) <= 1
    m = min(n, 30000)                       # every triangle for some rays, the binary nodes for all
    k = torch.randperm(n, generator=gen, device="cuda")[:m]
    brute = M.trace_anyhit(sc, o[:, k].contiguous(), d[:, k].contiguous(), brute=True)
    assert torch.equal(hit[k], brute)
    assert np.array_equal(to_np(hit), to_np(M.trace_anyhit(sc, o, d, mode="binary")))
    assert torch.equal(hit, M.trace_anyhit(sc, o, d, mode="wide"))
