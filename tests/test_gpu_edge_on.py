"""Triangles seen edge on, in front of a wall, against the oracle: planes
exactly through the camera centre have no depth, and on planes a micrometre
off it the pixel centres beside the triangle's line lie behind the camera
(1/z < 0).  The oracle ignores such fragments.  The images and records must
also not depend on which triangles share a wave (a few larger triangles among
the small ones send whole waves another way), on the tile shape, or on whether
records are cut into slices."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (integer principal point and equal focal lengths: the line y = x/2 runs through the centres of pixels (cx + 2k, cy + k))
CAM = S.Camera(64.0, 64.0, 48.0, 35.0, 97, 71, 0.1, 16.0)
T = np.eye(4)[:3]
N = 3000


def _mesh(off, size, beside):
    """A wall at z = 12, N triangles of `size` px on the plane y = x/2 + off, and with `beside` a 4 px triangle behind
    the wall after every 20 of them."""
    rng = np.random.default_rng(17)
    z = np.exp(rng.uniform(np.log(0.5), np.log(10.0), (N, 3)))
    du = 2.0 * rng.integers(-20, 21, (N, 1)) + rng.uniform(-0.5 * size, 0.5 * size, (N, 3))
    x = (du / CAM.fx * z).astype(np.float32)
    P = np.stack([x, (0.5 * x + np.float32(off)).astype(np.float32), z.astype(np.float32)], -1)
    if beside:
        c = np.stack([rng.uniform(4, 92, N // 20), rng.uniform(4, 66, N // 20)], -1)[:, None]
        px = c + np.array([[-2.0, -2.0], [2.0, -2.0], [-2.0, 2.0]])
        q = np.concatenate([(px - [CAM.cx, CAM.cy]) / CAM.fx * 14.0, np.full((N // 20, 3, 1), 14.0)], -1).astype(np.float32)
        P = np.concatenate([P.reshape(N // 20, 20, 3, 3), q[:, None]], 1).reshape(-1, 3, 3)
    wall = np.array([[-40, -40, 12], [40, -40, 12], [40, 40, 12], [-40, -40, 12], [40, 40, 12], [-40, 40, 12]], np.float32)
    xyz = np.concatenate([wall, P.reshape(-1, 3)])
    tri = np.arange(len(xyz), dtype=np.int32).reshape(-1, 3)
    return xyz, tri, (np.arange(len(tri)) >= 2).astype(np.uint8)


@pytest.mark.parametrize("tile", [(64, 32), (8, 8)])
@pytest.mark.parametrize("beside", [False, True])
@pytest.mark.parametrize("off,size", [(0.0, 3.0), (0.0, 9.0), (1e-6, 3.0), (1e-6, 9.0), (-1e-6, 3.0)])
def test_edge_on_triangles_against_the_oracle(off, size, beside, tile):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_06813_amd as rm
    mesh = _mesh(off, size, beside)
    ref = O.render(mesh, CAM, T)
    assert (ref["ncov"] > 1).sum() > 30                     # edge-on triangles do cover pixel centres
    fl = O.flags(ref, CAM)
    ok = ~(fl["near_tie"] | fl["far_tie"])
    assert ok.mean() > 0.95
    m = rm.Mesh.from_arrays(*mesh).prepare()
    scan = rm.scan_image(torch.full((CAM.height, CAM.width), 11.9, device="cuda"), 0.5, 15.0, cam=CAM)
    Td = torch.from_numpy(T.reshape(1, 12).copy()).cuda()
    ctx = rm.context()
    ctx.set_tile(*tile)
    got = []
    try:
        for schedule in (1, 0, 0):
            ctx.set_schedule(schedule)
            r = rm.render_depth(m, CAM, Td)
            np.testing.assert_array_equal(r["tri"].cpu().numpy().reshape(-1)[ok], ref["id"][ok])
            assert torch.isfinite(r["depth"]).all()
            got.append([r["tri"], r["depth"].view(torch.int32), rm.align_cost(m, scan, Td, 0.3),
                        rm.align_cost_grad(m, scan, Td, 0.3)])
    finally:
        ctx.set_schedule(0)
        ctx.set_tile(0, 0)
    for other in got[1:]:
        for k, (a, b) in enumerate(zip(other, got[0])):
            assert torch.equal(a, b), k
