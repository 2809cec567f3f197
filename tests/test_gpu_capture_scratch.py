"""Capture of a call whose scratch was sized by another one: a call that fits the
scratch that is there without the slots of cut records is captured and
replayed with as many slots as are left (none, or a few), not refused."""
import numpy as np
import pytest

from gpu_helpers import EPS, oracle_map, workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_poses", [1, 3])
@pytest.mark.parametrize("tile", [(64, 32), (16, 16)])
@pytest.mark.parametrize("sizing_cap", [64, 1024])
def test_capture_in_scratch_without_room_for_all_slots(sizing_cap, tile, n_poses, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_06813_amd as rm
    from paper_1702_06813_amd import rendermap
    w = workload("kinect")
    mesh = rm.Mesh.from_arrays(*oracle_map("kinect")).prepare()
    scan = rm.scan_image(torch.from_numpy(w.scan_depth).cuda(), cam=w.cam)
    T = torch.from_numpy(np.ascontiguousarray(w.poses[:n_poses].reshape(-1, 12))).cuda()
    ctx = rm.Context(0)                        # its scratch starts empty
    monkeypatch.setitem(rendermap._ctxs, 0, ctx)
    ctx.set_tile(*tile)
    ctx.set_bin_pool(0)
    ctx.set_bin_cap(sizing_cap)
    ctx.set_schedule(1)                        # cuts no records: scratch without slots
    ref = rm.align_cost_grad(mesh, scan, T, EPS)
    out = torch.empty_like(ref)
    ctx.set_schedule(0)
    ctx.set_bin_cap(64)                        # the bins shrink: the rest may hold slots
    with rm.Graph(torch.device("cuda", 0)) as g:
        rm.align_cost_grad(mesh, scan, T, EPS, out=out)
    for _ in range(3):
        out.fill_(float("nan"))
        g.replay()
        assert torch.equal(out, ref)
    torch.cuda.synchronize()
    del g
