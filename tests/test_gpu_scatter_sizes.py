"""The probe gradient where its sums change their workgroup: a probe past 4M
texels (48 KB of sums) and the bilinear taps (96 KB), against the oracle with
the backward parity test's tolerances."""

import numpy as np
import pytest

from workloads import make_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,bilinear", [(2049, 2050, False), (31, 67, True), (3, 5, True)])
def test_scatter_sizes(H, W, bilinear):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_03380_amd as M
    from tests.test_gpu_parity import _bwd_parity
    w = make_workload("tiny")
    r = np.random.Generator(np.random.PCG64(H + W))
    w.env = r.lognormal(0, 1, (H, W, 3)).astype(np.float32)
    _bwd_parity(w, flags=M.FLAG_BILINEAR if bilinear else 0)
