"""Probe tables at the edges of their kernels (the scan's steps of 16, four
texels a lane across row ends, the largest sides) against the oracle's, with
the tolerance of the bitwise table test: one FP32 ulp, rarely."""

import numpy as np
import pytest

import oracle
from tests.parity_util import to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(1, 1), (1, 2), (2, 3), (3, 15), (5, 16), (7, 17), (31, 33), (16, 47), (3, 4096),
                                 (4096, 3), (333, 1025)])
def test_env_tables_sizes(H, W):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_03380_amd as M
    r = np.random.Generator(np.random.PCG64(H * 5000 + W))
    e = r.lognormal(0, 2, (H, W, 3)).astype(np.float32)
    e[r.random((H, W)) < 0.2] = 0.0
    if not e.any():
        e[0, 0] = 1.0
    got = [to_np(t) for t in M.Env(torch.from_numpy(e).cuda()).tables()]
    ref = oracle.EnvTables(e)
    for a, b in zip(got, (ref.cond, ref.marg, ref.pdf)):
        diff = np.abs(a.view(np.uint32).astype(np.int64) - b.reshape(a.shape).view(np.uint32).astype(np.int64))
        assert diff.max() <= 1 and (diff != 0).sum() <= max(2, a.size // 100000)
