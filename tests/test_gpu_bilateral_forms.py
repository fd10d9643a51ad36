"""The denoiser's launches of many tiles against launches of few: views are
independent, so a batch on one side of a form's tile count has to give what its
views give one at a time on the other (each form is within the parity tests'
bound of the oracle, so the two are within twice that)."""

import pytest

from oracle import bilateral as B
from tests.test_bilateral import TOL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# tiles of one view (of 16 x 16 pixels, the last row and column ragged) and views
@pytest.mark.parametrize("nc,sigma,ty,tx,views", [(6, 2.0, 16, 16, 3), (3, 2.0, 19, 27, 1), (6, 2.6, 8, 16, 3),
                                                 (6, 2.3, 16, 16, 3), (1, 2.6, 16, 17, 2)])
def test_many_tiles(nc, sigma, ty, tx, views):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_03380_amd as M
    H, W = 16 * ty - 5, 16 * tx - 3
    gen = torch.Generator(device="cuda").manual_seed(nc * 100 + ty)
    n = views * H * W
    r = lambda *s: torch.rand(s, generator=gen, device="cuda")  # noqa: E731
    depth = 2 + 0.3 * r(n)
    nrm = torch.stack([0.4 * r(n) - 0.2, 0.4 * r(n) - 0.2, torch.ones(n, device="cuda")])
    mask = (r(n) < 0.9).to(torch.uint8)
    x, g = r(nc, n), r(nc, n)
    whole = M.BilateralGuide(depth, nrm, mask, views, H, W, sigma)
    out, wsum = M.bilateral_fwd(whole, x)
    gin = M.bilateral_bwd(whole, g, wsum)
    R = B.radius(sigma)
    rows = [(v, 0, H) for v in range(views)] if views > 1 else [(0, 0, H // 2), (0, H // 2, H)]
    for v, y0, y1 in rows:
        # a part with the rows its footprint (of the adjoint: twice that, one
        # more for the depth gradient) reaches
        m = 2 * R + 1
        a, b = max(0, y0 - m), min(H, y1 + m)
        part = lambda t: t.reshape(-1, views, H, W)[:, v, a:b].reshape(t.shape[:-1] + (-1,)).contiguous()  # noqa: E731
        guide = M.BilateralGuide(part(depth), part(nrm), part(mask), 1, b - a, W, sigma)
        o, w = M.bilateral_fwd(guide, part(x))
        gi = M.bilateral_bwd(guide, part(g), w)
        keep = slice((y0 - a) * W, (y1 - a) * W)
        assert (o - part(out))[:, keep].abs().max() <= 2 * TOL
        scale = M.bilateral_bwd(guide, part(g).abs(), w)[:, keep]
        assert ((gi - part(gin))[:, keep].abs() <= 2 * TOL * scale + 1e-6).all()
