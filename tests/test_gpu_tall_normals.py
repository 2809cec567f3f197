"""Normals of depth images with very many rows (rm_depth_normals takes any
height whose pixels number at most 2^26): against a plain float64 evaluation
at the first and last rows and across the image."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(524_288, 5), (524_289, 5), (600_000, 33), (3, 700_000)])
def test_normals_of_tall_and_wide_images(H, W):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_06813_amd as rm
    rng = np.random.default_rng(H + W)
    z = (2.0 + 0.05 * rng.standard_normal((H, W))).astype(np.float32)
    z[rng.random((H, W)) < 0.01] = np.nan
    cam = S.Camera(500.0, 510.0, 0.5 * (W - 1), 0.5 * (H - 1), W, H)
    got = rm.depth_normals(torch.from_numpy(z).cuda(), cam, 1.0, 1).cpu().numpy()
    for y0 in sorted({0, max(0, H // 2 - 20), max(0, H - 40)}):
        for x0 in sorted({0, max(0, W // 2 - 20), max(0, W - 40)}):
            y1, x1 = min(H, y0 + 40), min(W, x0 + 40)
            ya, yb, xa, xb = max(0, y0 - 2), min(H, y1 + 2), max(0, x0 - 2), min(W, x1 + 2)
            sub = S.Camera(500.0, 510.0, 0.0, 0.0, xb - xa, yb - ya)
            want = O.depth_normals(z[ya:yb, xa:xb], sub, 1.0, 1)[y0 - ya:y1 - ya, x0 - xa:x1 - xa]
            have = got[y0:y1, x0:x1]
            # (the piece's own border is the image's where they meet, else cut off above)
            np.testing.assert_array_equal(np.isnan(have), np.isnan(want))
            assert np.nanmax(np.abs(have - want), initial=0.0) < 1e-6
