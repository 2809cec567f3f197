"""Unions of no, one, two and more meshes: indices offset by the vertices before
them, tensors of their own, the same error for a union of nothing."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


def _parts(Mesh, n):
    rng = np.random.default_rng(n)
    parts = []
    for k in range(n):
        t = rng.integers(0, 4 + k, (3 + 2 * k, 3)).astype(np.int32)
        parts.append(Mesh.from_arrays(rng.standard_normal((4 + k, 3)).astype(np.float32), t,
                                      rng.integers(0, 2, len(t)).astype(np.uint8), device="cpu"))
    return parts


@pytest.mark.parametrize("n", [1, 2, 3, 5])
def test_union(n):
    from paper_1702_06813_amd.rendermap import Mesh
    parts = _parts(Mesh, n)
    before = [p.tri.clone() for p in parts]
    off = np.concatenate([[0], np.cumsum([len(p.xyz) for p in parts])])
    m = Mesh.concat(parts)
    np.testing.assert_array_equal(m.tri, np.concatenate([b.numpy() + o for b, o in zip(before, off)]))
    np.testing.assert_array_equal(m.xyz, torch.cat([p.xyz for p in parts]))
    assert m.tri.dtype == torch.int32
    m.tri.fill_(-1)
    for p, b in zip(parts, before):
        assert torch.equal(p.tri, b)


def test_union_of_nothing():
    from paper_1702_06813_amd.rendermap import Mesh
    with pytest.raises(ValueError):
        Mesh.concat([])
