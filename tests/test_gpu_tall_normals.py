"""Normals of long depth images (rm_depth_normals takes any size up to 2^26
pixels), in one launch and in two: against the oracle in float64 at the first
and last rows and across the image, and captured without scratch."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# (from 65,536 pixels on: less than 8 pixels wide two launches, less than 24 wide or 8 high two with a radius above 2)
@pytest.mark.parametrize("H,W,R", [(524_288, 9, 1), (524_289, 9, 1), (600_000, 33, 1), (600_000, 33, 4), (524_289, 5, 1),
                                   (9_363, 7, 0), (9_362, 7, 8), (4_000, 23, 2), (4_000, 23, 3), (4_000, 24, 3),
                                   (3, 700_000, 2), (3, 700_000, 3), (7, 12_000, 8), (8, 12_000, 8), (70_000, 1, 4)])
def test_normals_of_tall_and_wide_images(H, W, R):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_06813_amd as rm
    rng = np.random.default_rng(H + W)
    z = (2.0 + 0.05 * rng.standard_normal((H, W))).astype(np.float32)
    z[rng.random((H, W)) < 0.01] = np.nan
    cam = S.Camera(500.0, 510.0, 0.5 * (W - 1), 0.5 * (H - 1), W, H)
    got = rm.depth_normals(torch.from_numpy(z).cuda(), cam, 1.0, R).cpu().numpy()
    for y0 in sorted({0, max(0, H // 2 - 20), max(0, H - 40)}):
        for x0 in sorted({0, max(0, W // 2 - 20), max(0, W - 40)}):
            y1, x1 = min(H, y0 + 40), min(W, x0 + 40)
            ya, yb, xa, xb = max(0, y0 - R - 1), min(H, y1 + R + 1), max(0, x0 - R - 1), min(W, x1 + R + 1)
            sub = S.Camera(500.0, 510.0, 0.0, 0.0, xb - xa, yb - ya)
            want = O.depth_normals(z[ya:yb, xa:xb], sub, 1.0, R)[y0 - ya:y1 - ya, x0 - xa:x1 - xa]
            have = got[y0:y1, x0:x1]
            # (the piece's own border is the image's where they meet, else cut off above)
            np.testing.assert_array_equal(np.isnan(have), np.isnan(want))
            assert np.nanmax(np.abs(have - want), initial=0.0) < 1e-6


@pytest.mark.parametrize("scratch", [False, True])
def test_capture_of_a_narrow_image(scratch, monkeypatch):
    """Where scratch cannot grow the one-launch form takes over, with the same normals."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_06813_amd as rm
    from paper_1702_06813_amd import rendermap
    H, W = 20_000, 6
    z = torch.from_numpy((2.0 + 0.05 * np.random.default_rng(1).standard_normal((H, W))).astype(np.float32)).cuda()
    want = rm.depth_normals(z, S.Camera(500.0, 510.0, 2.5, 9999.5, W, H), 1.5, 3)
    monkeypatch.setitem(rendermap._ctxs, 0, rm.Context(0))
    got = torch.empty_like(want)

    def call():
        rm.context().call("rm_depth_normals", rendermap._ptr(z), H, W, 500.0, 510.0, 1.5, 3, rendermap._ptr(got))

    if scratch:
        call()
    with rm.Graph(torch.device("cuda", 0)) as g:
        call()
    for _ in range(3):
        got.fill_(0.0)
        g.replay()
        assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    torch.cuda.synchronize()
    del g
