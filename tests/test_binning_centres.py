"""Triangles that binning leaves out because they cover no pixel centre (CPU).

Emulates the rule in numpy (float32 footprint, margin of 1/64 px plus the
bound on the camera centre's rounding; no centre in the box, or a single one
that lies outside an edge of an area of certain sign) on triangles of 0.02 to 4 px and checks with the
contract's integer edge functions that none of the left-out ones covers a
centre, at two image sizes on scenes placed up to 1e6 m from the world origin;
and on the GPU renders a wall meshed below the pixel size without a hole."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import scenes as S

from test_binning_margin import _f32, _footprint

CAM = S.Camera(262.5, 250.0, 79.5, 59.25, 160, 120, z_near=0.1, z_far=16.0)
LARGE = S.Camera(1050.0, 1043.0, 639.5, 479.25, 1280, 960, z_near=0.1, z_far=20.0)


def _misses(u, v, m):
    """misses_centres of the footprint polygons [N, 4] in float32."""
    u, v = _f32(u), _f32(v)
    umin, umax, vmin, vmax = u.min(1), u.max(1), v.min(1), v.max(1)
    x0, x1, y0, y1 = np.ceil(_f32(umin - m)), np.floor(_f32(umax + m)), np.ceil(_f32(vmin - m)), np.floor(_f32(vmax + m))
    none = ((x0 > x1) | (y0 > y1)) & (umax - umin + vmax - vmin < 4.0)
    j = [1, 2, 3, 0]
    d = lambda a, i: _f32(a[:, i] - a[:, 0])
    cross = lambda i, k: _f32(_f32(d(u, i) * d(v, k)) - _f32(d(v, i) * d(u, k)))
    area2 = _f32(cross(1, 2) + cross(2, 3))
    L = _f32(_f32(umax - umin) + _f32(vmax - vmin))
    sg = np.where(area2 > 0, 1.0, -1.0)[:, None]
    A, B = -sg * _f32(v[:, j] - v), sg * _f32(u[:, j] - u)
    dx, dy = _f32(x0[:, None] - u), _f32(y0[:, None] - v)
    out = (_f32(A * dx + B * dy) < -m[:, None] * (np.abs(A) + np.abs(B) + 2 * (np.abs(dx) + np.abs(dy)))).any(1)
    return none | ((x0 == x1) & (y0 == y1) & (np.abs(area2) > 2 * m * (L + m)) & out)


def _covers(sub):
    """Whether snapped triangles [N, 6] (1/256 px) cover a pixel centre (top-left rule, y down)."""
    X, Y = sub[:, 0::2].copy(), sub[:, 1::2].copy()
    area = (X[:, 1] - X[:, 0]) * (Y[:, 2] - Y[:, 0]) - (Y[:, 1] - Y[:, 0]) * (X[:, 2] - X[:, 0])
    f = area < 0
    X[f], Y[f] = X[f][:, [0, 2, 1]], Y[f][:, [0, 2, 1]]
    px, py = -(-X.min(1) // 256), -(-Y.min(1) // 256)
    hit = np.zeros(len(sub), bool)
    for oy in range(7):
        for ox in range(7):
            x, y = 256 * (px + ox), 256 * (py + oy)
            inside = area != 0
            for k in range(3):
                dx, dy = X[:, (k + 1) % 3] - X[:, k], Y[:, (k + 1) % 3] - Y[:, k]
                top = (dy < 0) | ((dy == 0) & (dx > 0))
                inside &= dx * (y - Y[:, k]) - dy * (x - X[:, k]) - np.where(top, 0, 1) >= 0
            hit |= inside
    return hit


@pytest.mark.parametrize("cam", [CAM, LARGE], ids=["160x120", "1280x960"])
@pytest.mark.parametrize("scale", [0.0, 1e3, 1e5, 1e6])
def test_left_out_triangles_cover_no_centre(scale, cam):
    rng = np.random.default_rng(int(scale) % 1000 + 5)
    n = 60000
    z = np.exp(rng.uniform(np.log(0.15), np.log(15.0), n))
    size = np.exp(rng.uniform(np.log(0.02), np.log(4.0), n))
    c = np.stack([rng.uniform(-2, cam.width + 2, n), rng.uniform(-2, cam.height + 2, n)], 1)
    c[::3] = np.round(c[::3])                               # many near centres
    px = c[:, None] + size[:, None, None] * rng.uniform(-0.5, 0.5, (n, 3, 2))
    zz = z[:, None] * (1 + 0.02 * rng.standard_normal((n, 3)))
    P = np.stack([(px[..., 0] - cam.cx) / cam.fx * zz, (px[..., 1] - cam.cy) / cam.fy * zz, zz], -1).reshape(-1, 3)
    T = np.array(S.look_pose(np.array([1.0, -0.7, 0.3]), 0.7, 0.2, 0.1), np.float64)
    T[:3, 3] += scale * np.array([1.0, -0.7, 0.3])
    xyz = (P @ T[:3, :3].T + T[:3, 3]).astype(np.float32)
    mesh = (xyz, np.arange(3 * n, dtype=np.int32).reshape(n, 3), np.zeros(n, np.uint8))
    Z, u, v, dn, tn = _footprint(xyz, T, cam)
    Z, u, v, dn = (a.reshape(n, 3) for a in (Z, u, v, dn))
    ok = (Z > cam.z_near * 1.01).all(1)
    m = 1 / 64 + 2.0 ** -23 * (tn + 9 * dn.max(1)) * (max(cam.fx, cam.fy) + cam.width) / np.maximum(Z.min(1), cam.z_near)
    poly = [0, 1, 2, 2]
    left = np.zeros(n, bool)
    left[ok] = _misses(u[ok][:, poly], v[ok][:, poly], m[ok])
    sub = O.contract_subtriangles(mesh, cam, T)
    covering = np.unique(sub[:, 0][_covers(sub[:, 1:])])
    assert not left[covering].any(), int(left[covering].sum())
    if scale == 0.0:
        assert left.mean() > 0.2                            # the rule has something to do


@pytest.mark.gpu
@pytest.mark.parametrize("z,cell", [(15.0, 0.018), (15.5, 0.012), (6.0, 0.006)])
def test_a_wall_meshed_below_the_pixel_size_has_no_holes(z, cell):
    """1280x960 pixels of a tilted wall of right triangles of 1.3, 0.8 and 1.0 px: every pixel
    is covered, at the plane's depth (float32 depth and vertices: 1e-5 of z)."""
    import torch
    import paper_1702_06813_amd as rm
    nx, ny = int(1.35 * z / cell), int(1.05 * z / cell)
    x = (np.arange(nx + 1) - nx / 2) * cell
    y = (np.arange(ny + 1) - ny / 2) * cell
    X, Y = np.meshgrid(x, y)
    xyz = np.stack([X, Y, z + 0.05 * X - 0.03 * Y], -1).reshape(-1, 3).astype(np.float32)
    q = (np.arange(ny)[:, None] * (nx + 1) + np.arange(nx)).ravel()
    tri = np.concatenate([np.stack([q, q + 1, q + nx + 1], 1), np.stack([q + 1, q + nx + 2, q + nx + 1], 1)])
    mesh = rm.Mesh(torch.from_numpy(xyz).cuda(), torch.from_numpy(tri.astype(np.int32)).cuda(),
                   torch.zeros(len(tri), dtype=torch.uint8, device="cuda"))
    depth = rm.render_depth(mesh, LARGE, torch.eye(4, dtype=torch.float64, device="cuda")[:3].reshape(1, 12))["depth"][0].double().cpu().numpy()
    u, v = np.meshgrid(np.arange(1280), np.arange(960))
    rx, ry = (u - LARGE.cx) / LARGE.fx, (v - LARGE.cy) / LARGE.fy
    exact = z / (1 - 0.05 * rx + 0.03 * ry)
    assert np.isfinite(depth).all(), int((~np.isfinite(depth)).sum())
    assert np.abs(depth - exact).max() < 1e-5 * z
