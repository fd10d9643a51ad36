"""Exact boxes, links and leaf coverage of the BVH on meshes around the edges of
the fitting blocks (256 triangles) and super-blocks (256 blocks)."""

import numpy as np
import pytest

from tests.parity_util import to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt", [2, 3, 256, 257, 513, 65535, 65536, 65537, 65793, 131073, 200000])
def test_bvh_sizes(nt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_03380_amd as M
    r = np.random.Generator(np.random.PCG64(nt))
    v = (r.uniform(-1, 1, (nt, 1, 3)) + 0.01 * r.normal(size=(nt, 3, 3))).astype(np.float32).reshape(-1, 3)
    f = np.arange(3 * nt, dtype=np.int32).reshape(nt, 3)
    sc = M.Scene(torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda())
    info = sc.info()
    nodes, tris = (to_np(t) for t in sc.nodes())
    esc, pay = nodes[:, 3], nodes[:, 7]
    lo, hi = (np.ascontiguousarray(nodes[:, k:k + 3]).view(np.float32) for k in (0, 4))
    assert esc[0] == len(nodes) == info["n_nodes"]
    leaf = np.nonzero(pay != 0)[0]
    assert (esc[leaf] == leaf + 1).all()
    first, cnt = pay[leaf] >> 3, pay[leaf] & 7
    assert first[0] == 0 and (first[1:] == (first + cnt)[:-1]).all() and first[-1] + cnt[-1] == nt
    tlo, thi = tris[:, :, :3].min(1), tris[:, :, :3].max(1)
    ends = first + cnt
    for k in range(int(cnt.max())):
        at = np.minimum(first + k, ends - 1)
        lo_k = tlo[at] if k == 0 else np.minimum(lo_k, tlo[at])
        hi_k = thi[at] if k == 0 else np.maximum(hi_k, thi[at])
    assert np.array_equal(lo[leaf], lo_k) and np.array_equal(hi[leaf], hi_k)
    inner = np.nonzero(pay == 0)[0]
    a, b = inner + 1, esc[inner + 1]
    assert (b < esc[inner]).all() and (esc[b] == esc[inner]).all()
    assert np.array_equal(lo[inner], np.minimum(lo[a], lo[b])) and np.array_equal(hi[inner], np.maximum(hi[a], hi[b]))
    depth = np.zeros(len(nodes), np.int64)
    for i in inner:                                   # pre-order: parents first
        depth[i + 1] = depth[esc[i + 1]] = depth[i] + 1
    assert info["max_depth"] == depth.max()
    area = lambda x: 2 * (x[:, 0] * x[:, 1] + x[:, 1] * x[:, 2] + x[:, 2] * x[:, 0])  # noqa: E731
    ext = hi.astype(np.float64) - lo
    dc = area(ext[leaf]).sum() / area(ext[:1])[0]
    assert abs(info["depth_complexity"] - dc) <= 1e-6 * dc
    # the input triangles, each once
    key = lambda x: x[np.lexsort(x.T[::-1])]  # noqa: E731
    assert np.array_equal(key(v[f].reshape(nt, 9)), key(tris[:, :, :3].reshape(nt, 9)))
