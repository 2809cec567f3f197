"""Triangles that binning leaves out because they cover no pixel centre (CPU).

Emulates the rule in numpy (float32 footprint, margin of 1/64 px plus the
bound on the camera centre's rounding; no centre in the box, or a single one
that lies outside an edge) on triangles of 0.02 to 4 px and checks with the
contract's integer edge functions that none of the left-out ones covers a
centre, on scenes placed up to 1e6 m from the world origin."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import scenes as S

from test_binning_margin import _f32, _footprint

CAM = S.Camera(262.5, 250.0, 79.5, 59.25, 160, 120, z_near=0.1, z_far=16.0)


def _misses(u, v, m):
    """misses_centres of the footprint polygons [N, 4] in float32."""
    u, v = _f32(u), _f32(v)
    umin, umax, vmin, vmax = u.min(1), u.max(1), v.min(1), v.max(1)
    x0, x1, y0, y1 = np.ceil(_f32(umin - m)), np.floor(_f32(umax + m)), np.ceil(_f32(vmin - m)), np.floor(_f32(vmax + m))
    none = ((x0 > x1) | (y0 > y1)) & (umax - umin + vmax - vmin < 4.0)
    j = [1, 2, 3, 0]
    area2 = _f32(u * v[:, j] - u[:, j] * v).sum(1)
    sg = np.where(area2 > 0, 1.0, -1.0)[:, None]
    A, B = -sg * _f32(v[:, j] - v), sg * _f32(u[:, j] - u)
    dx, dy = _f32(x0[:, None] - u), _f32(y0[:, None] - v)
    out = (_f32(A * dx + B * dy) < -m[:, None] * (np.abs(A) + np.abs(B) + 2 * (np.abs(dx) + np.abs(dy)))).any(1)
    return none | ((x0 == x1) & (y0 == y1) & (np.abs(area2) >= 1e-3) & out)


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


@pytest.mark.parametrize("scale", [0.0, 1e3, 1e5, 1e6])
def test_left_out_triangles_cover_no_centre(scale):
    rng = np.random.default_rng(int(scale) % 1000 + 5)
    n = 60000
    z = np.exp(rng.uniform(np.log(0.15), np.log(15.0), n))
    size = np.exp(rng.uniform(np.log(0.02), np.log(4.0), n))
    c = np.stack([rng.uniform(-2, 162, n), rng.uniform(-2, 122, n)], 1)
    c[::3] = np.round(c[::3])                               # many near centres
    px = c[:, None] + size[:, None, None] * rng.uniform(-0.5, 0.5, (n, 3, 2))
    zz = z[:, None] * (1 + 0.02 * rng.standard_normal((n, 3)))
    P = np.stack([(px[..., 0] - CAM.cx) / CAM.fx * zz, (px[..., 1] - CAM.cy) / CAM.fy * zz, zz], -1).reshape(-1, 3)
    T = np.array(S.look_pose(np.array([1.0, -0.7, 0.3]), 0.7, 0.2, 0.1), np.float64)
    T[:3, 3] += scale * np.array([1.0, -0.7, 0.3])
    xyz = (P @ T[:3, :3].T + T[:3, 3]).astype(np.float32)
    mesh = (xyz, np.arange(3 * n, dtype=np.int32).reshape(n, 3), np.zeros(n, np.uint8))
    Z, u, v, dn, tn = _footprint(xyz, T, CAM)
    Z, u, v, dn = (a.reshape(n, 3) for a in (Z, u, v, dn))
    ok = (Z > CAM.z_near * 1.01).all(1)
    m = 1 / 64 + 2.0 ** -23 * (tn + 9 * dn.max(1)) * (max(CAM.fx, CAM.fy) + 160) / np.maximum(Z.min(1), CAM.z_near)
    poly = [0, 1, 2, 2]
    left = np.zeros(n, bool)
    left[ok] = _misses(u[ok][:, poly], v[ok][:, poly], m[ok])
    sub = O.contract_subtriangles(mesh, CAM, T)
    covering = np.unique(sub[:, 0][_covers(sub[:, 1:])])
    assert not left[covering].any(), int(left[covering].sum())
    if scale == 0.0:
        assert left.mean() > 0.2                            # the rule has something to do
