"""Meshing at the edges of its 8x8 blocks of quads: grids of one row or column,
of exactly one block, one node more and one less, against the oracle,
bit for bit."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("radius", [0, 1, 16])
@pytest.mark.parametrize("size", [(1, 9), (9, 1), (2, 2), (8, 8), (9, 9), (10, 17), (17, 10), (33, 65)])
def test_block_edges_bitexact(size, radius):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_06813_amd as rm
    H, W = size
    rng = np.random.default_rng(H * 100 + W)
    z = (2.0 * (1 + 0.02 * rng.standard_normal((H, W)))).astype(np.float32)
    z[rng.random((H, W)) < 0.1] = 0.0
    z[rng.random((H, W)) < 0.1] = np.nan
    z[rng.random((H, W)) < 0.1] *= 3
    cam = S.Camera(40.0, 40.0, 0.5 * (W - 1), 0.5 * (H - 1), W, H)
    T = S.look_pose(np.array([0.3, -0.2, 1.0]), 0.4, 0.1)
    ref = O.meshify(z, cam, T, 1, smooth_radius=radius)
    m = rm.mesh_from_range(torch.from_numpy(z).cuda(), cam, T, 1, smooth_radius=radius)
    for got, want in zip((m.xyz, m.tri, m.cls), ref):
        np.testing.assert_array_equal(got.cpu().numpy(), want)
