"""Cameras with mirrored axes (negative focal lengths): two parallel slanted
walls a fraction of a pixel's slope apart, the nearer one meshed below the
pixel size with its triangles in random order, so that its clusters reach far
and are drawn after the wall behind.  Each of its triangles lies in front of
what is drawn by then, and none may be taken for hidden."""
import numpy as np
import pytest

from workloads import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

W, H, Z0, SLOPE, GAP, CELL = 320, 240, 5.0, 0.8, 6e-4, 0.0125


def _wall(scale, order=None):
    """Points (x, y, Z0 + SLOPE x) scaled towards the camera, in a 5.4 m x 4.4 m grid of right triangles."""
    nx, ny = int(5.4 / CELL), int(4.4 / CELL)
    X, Y = np.meshgrid((np.arange(nx + 1) - nx / 2) * CELL, (np.arange(ny + 1) - ny / 2) * CELL)
    xyz = (np.stack([X, Y, Z0 + SLOPE * X], -1).reshape(-1, 3) * scale).astype(np.float32)
    q = (np.arange(ny)[:, None] * (nx + 1) + np.arange(nx)).ravel()
    tri = np.concatenate([np.stack([q, q + 1, q + nx + 1], 1), np.stack([q + 1, q + nx + 2, q + nx + 1], 1)])
    return xyz, tri if order is None else tri[order.permutation(len(tri))]


@pytest.mark.parametrize("fx,fy", [(300.0, 300.0), (-300.0, 300.0), (300.0, -300.0), (-300.0, -300.0)])
def test_the_nearer_of_two_close_walls_wins(fx, fy):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_06813_amd as rm
    # (1/z at the image's far side, x = 2.7 m, is 0.14, a pixel's slope 5.3e-4, the gap GAP / z = 8.4e-5)
    cam = S.Camera(fx, fy, 0.5 * (W - 1), 0.5 * (H - 1), W, H, z_near=0.1, z_far=20.0)
    far_xyz, far_tri = _wall(1.0)
    near_xyz, near_tri = _wall(1.0 - GAP, np.random.default_rng(3))
    xyz = np.concatenate([far_xyz, near_xyz])
    tri = np.concatenate([far_tri, near_tri + len(far_xyz)]).astype(np.int32)
    mesh = rm.Mesh.from_arrays(xyz, tri, np.zeros(len(tri), np.uint8)).prepare()
    T = torch.eye(4, dtype=torch.float64, device="cuda")[:3].reshape(1, 12).repeat(16, 1)
    ctx = rm.context()
    ctx.set_schedule(1)                        # a tile's triangles all by one workgroup: the far wall is whole first
    try:
        ids = rm.render_depth(mesh, cam, T)["tri"].cpu().numpy()
    finally:
        ctx.set_schedule(0)
    u = (np.arange(W) - cam.cx) / cam.fx
    v = (np.arange(H) - cam.cy) / cam.fy
    z = Z0 / (1 - SLOPE * u)
    inside = (np.abs(u * z) < 2.6)[None, :] & (np.abs(v[:, None] * z[None, :]) < 2.1)
    assert inside.mean() > 0.5
    assert (ids[:, inside] >= len(far_tri)).all(), int((ids[:, inside] < len(far_tri)).sum())
