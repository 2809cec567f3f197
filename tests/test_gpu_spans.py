"""Row spans of the tile rasterizer against the oracle's edge functions:
vertices and edges on pixel centres, horizontal edges, slivers, and vertices
around and beyond the distance up to which spans come from FP64 crossings
(32768 px from the tile), where the exact integer path takes over."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CAM = S.Camera(64.0, 64.0, 40.0, 33.0, 97, 71, 0.1, 16.0)
T = np.eye(4)[:3]


def _vertices(kind, rng, n):
    """[n, 3, 2] pixel positions, multiples of 1/256 px."""
    if kind == "centres":                      # whole and half pixels, many horizontal and vertical edges
        return rng.integers(-20, 240, (n, 3, 2)) / 2.0
    p = np.round(rng.uniform(-10, 110, (n, 3, 2)) * 256) / 256
    if kind == "slivers":                      # third vertex within 2/256 px of the first edge
        t = rng.uniform(0, 1, (n, 1))
        p[:, 2] = np.round((p[:, 0] + t * (p[:, 1] - p[:, 0])) * 256 + rng.integers(-2, 3, (n, 2))) / 256
    elif kind == "limit":                      # one vertex within 70 px of the span limit, seen from any tile
        p[:, 1, rng.integers(0, 2)] = rng.choice([-1, 1], n) * (32768 + rng.integers(-140, 141, n) / 2.0)
    elif kind == "far":                        # two vertices far outside, one on each side
        p[:, 1] = rng.integers(-100000, -33000, (n, 2))
        p[:, 2] = rng.integers(33000, 100000, (n, 2))
    return p


@pytest.mark.parametrize("tile", [(64, 32), (32, 32), (16, 16), (8, 8)])
@pytest.mark.parametrize("kind", ["centres", "fine", "slivers", "limit", "far"])
def test_row_spans_against_the_oracle(kind, tile):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_06813_amd as rm
    rng = np.random.default_rng(sum(map(ord, kind)))
    ctx = rm.context()
    Td = torch.from_numpy(T.reshape(1, 12).copy()).cuda()
    covered = flagged = 0
    ctx.set_tile(*tile)
    try:
        for _ in range(24):
            # one triangle at each power-of-two depth, so that positions project exactly
            z = np.array([1.0, 2.0, 4.0, 8.0])
            p = _vertices(kind, rng, 4)
            xyz = np.empty((4, 3, 3))
            xyz[..., 0] = (p[..., 0] - CAM.cx) / CAM.fx * z[:, None]
            xyz[..., 1] = (p[..., 1] - CAM.cy) / CAM.fy * z[:, None]
            xyz[..., 2] = z[:, None]
            mesh = (xyz.reshape(-1, 3).astype(np.float32), np.arange(12, dtype=np.int32).reshape(4, 3),
                    np.zeros(4, np.uint8))
            ref = O.render(mesh, CAM, T)
            got = rm.render_depth(rm.Mesh.from_arrays(*mesh).prepare(), CAM, Td)
            ids = got["tri"].cpu().numpy().reshape(-1)
            fl = O.flags(ref, CAM)
            ex = fl["near_tie"] | fl["far_tie"]
            np.testing.assert_array_equal(ids[~ex], ref["id"][~ex])
            covered += int((ref["id"] >= 0).sum())
            flagged += int(ex.sum())
    finally:
        ctx.set_tile(0, 0)
    assert covered > 0 and flagged == 0
