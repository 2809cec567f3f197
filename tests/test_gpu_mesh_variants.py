"""Every form of the meshing and normals kernels: windows of every kind of size
at strides above one on ragged images, their rows shared by eight lanes (up to
512 blocks of quads), two (up to 4,096) or one, grids without windows of as many
blocks as one workgroup takes whole (4,096) and more, normals of every radius;
and the union of meshes of which some are empty."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_06813_amd as rm
    return rm


def _depth(H, W):
    rng = np.random.default_rng(H * 1000 + W)
    z = (2.0 * (1 + 0.02 * rng.standard_normal((H, W)))).astype(np.float32)
    z[rng.random((H, W)) < 0.05] = 0.0
    z[rng.random((H, W)) < 0.05] = np.nan
    z[rng.random((H, W)) < 0.05] *= 3
    return z


def _mesh_bitexact(rm, H, W, stride, radius):
    z = _depth(H, W)
    cam = S.Camera(200.0, 210.0, 0.5 * (W - 1), 0.5 * (H - 1), W, H)
    T = S.look_pose(np.array([0.3, -0.2, 1.0]), 0.4, 0.1)
    ref = O.meshify(z, cam, T, stride, smooth_radius=radius)
    m = rm.mesh_from_range(torch.from_numpy(z).cuda(), cam, T, stride, smooth_radius=radius)
    for got, want in zip((m.xyz, m.tri, m.cls), ref):
        np.testing.assert_array_equal(got.cpu().numpy(), want)
    return len(ref[1])


@pytest.mark.parametrize("stride,radius", [(2, 3), (3, 16), (5, 0), (7, 15), (7, 16), (8, 11), (8, 12), (8, 16), (12, 4),
                                           (31, 2)])
@pytest.mark.parametrize("H,W", [(61, 190), (129, 67)])
def test_meshing_windows_bitexact(rm, H, W, stride, radius):
    assert _mesh_bitexact(rm, H, W, stride, radius) > 0


@pytest.mark.parametrize("radius", [0, 1, 2])
@pytest.mark.parametrize("H,W", [(129, 257), (137, 257), (513, 513), (513, 514)])
def test_meshing_block_offsets_bitexact(rm, H, W, radius):
    """16 x 32 = 512 blocks and 17 x 32, 64 x 64 = 4,096 and 64 x 65."""
    assert _mesh_bitexact(rm, H, W, 1, radius) > 30_000


@pytest.mark.parametrize("radius", range(9))
def test_normals_of_every_radius(rm, radius):
    """Against the oracle in 64 bits; float32 rounding of unit vectors, 6e-8."""
    for H, W in ((75, 101), (9, 33), (7, 5), (3, 3)):
        z = _depth(H, W)
        cam = S.Camera(200.0, 210.0, 0.5 * (W - 1), 0.5 * (H - 1), W, H)
        got = rm.depth_normals(torch.from_numpy(z).cuda(), cam, 1.5, radius).cpu().numpy()
        want = O.depth_normals(z, cam, 1.5, radius)
        np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
        if np.isfinite(want).any():
            assert np.nanmax(np.abs(got - want)) < 2e-7


@pytest.mark.parametrize("empty", [(), (0,), (2,), (4,), (0, 1), (1, 3, 4), (0, 1, 2, 3), (0, 1, 2, 3, 4)])
def test_union_with_empty_meshes(rm, empty):
    rng = np.random.default_rng(len(empty))
    xyz, tri, cls, off = [], [], [], 0
    parts = []
    for k in range(5):
        nt = 0 if k in empty else 5 + 3 * k
        v = rng.standard_normal((7 + k, 3)).astype(np.float32)
        t = rng.integers(0, 7 + k, (nt, 3)).astype(np.int32)
        c = rng.integers(0, 2, nt).astype(np.uint8)
        parts.append(rm.Mesh.from_arrays(v, t, c))
        xyz.append(v); tri.append(t + off); cls.append(c); off += len(v)
    m = rm.Mesh.concat(parts)
    assert m.tri.dtype == torch.int32 and m.tri.is_contiguous()
    for got, want in zip((m.xyz, m.tri, m.cls), (xyz, tri, cls)):
        np.testing.assert_array_equal(got.cpu().numpy(), np.concatenate(want))
