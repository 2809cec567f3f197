"""Cut records in calls that the three-launch order takes (more than 3,072
records) and where slots run out: the plan's log says how many slices the
records ask for, and records and images are bit-identical to the call with one
workgroup per record.  One pose looks at the map and the others away from it,
so that its records hold far more than a workgroup's share."""
import re

import numpy as np
import pytest

from gpu_helpers import EPS, workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _setup(n_away):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_06813_amd as rm
    w = workload("differentiation")
    mesh = rm.Mesh.concat([rm.mesh_from_range(torch.from_numpy(z).cuda(), w.cam, V, w.stride, w.z_min, w.z_max, w.max_edge,
                                              w.smooth_radius) for V, z in zip(w.views, w.view_depths)]).prepare()
    scan = rm.scan_image(torch.from_numpy(w.scan_depth).cuda(), cam=w.cam)
    away = np.array(w.poses[0], np.float64).reshape(3, 4).copy()
    away[:, 3] += 1000.0
    back = np.array(w.poses[0], np.float64).reshape(3, 4).copy()
    back[:, 3] -= 6.0 * back[:, 2]
    poses = np.concatenate([away.reshape(1, 12).repeat(n_away, 0), back.reshape(1, 12)])
    return rm, w, mesh, scan, torch.from_numpy(np.ascontiguousarray(poses)).cuda()


def _slots(capfd):
    """(slices asked for, slots there, scratch bytes) of the last plan in the log."""
    found = re.findall(r"cut records ask for (\d+) of (\d+) slice slots, (\d+) bytes", capfd.readouterr().err)
    assert found
    return tuple(int(x) for x in found[-1])


# 640x480: 1,200 tiles of 16x16, 300 of 32x32, 150 of 64x32
@pytest.mark.parametrize("tile,n_away", [((16, 16), 0), ((16, 16), 2), ((16, 16), 5), ((32, 32), 9), ((32, 32), 10),
                                         ((64, 32), 19), ((64, 32), 20), ((64, 32), 53)])
def test_cut_records_of_large_calls(tile, n_away, capfd, monkeypatch):
    rm, w, mesh, scan, T = _setup(n_away)
    from paper_1702_06813_amd import rendermap
    monkeypatch.setitem(rendermap._ctxs, 0, rm.Context(0))
    monkeypatch.setenv("RM_LOG", "1")
    ctx = rm.context()
    ctx.set_tile(*tile)
    vn = torch.nn.functional.normalize(torch.randn(mesh.xyz.shape, generator=torch.Generator().manual_seed(3))).cuda()
    got = {}
    for schedule in (1, 0, 0):
        ctx.set_schedule(schedule)
        ctx.set_bin_cap(0)                     # the next call sizes its bins again and logs its plan
        capfd.readouterr()
        now = [rm.align_cost_grad(mesh, scan, T, EPS)]
        asked, there, _ = _slots(capfd)
        if schedule == 1:
            assert (asked, there) == (0, 0)
        else:
            assert 0 < asked <= there
        r = rm.render_depth(mesh, w.cam, T)
        now += [rm.align_cost(mesh, scan, T, EPS), rm.icp_cost_grad(mesh, scan, T, vn), r["tri"],
                r["depth"].view(torch.int32)]
        for k, x in enumerate(now):
            assert torch.equal(x, got.setdefault(k, x.clone())), (schedule, k)


@pytest.mark.parametrize("n_away", [0, 22])
def test_more_slices_than_slots(n_away, capfd, monkeypatch):
    """The capture's scratch was sized without slots: what is left of it holds some, fewer than the records ask for."""
    rm, w, mesh, scan, T = _setup(n_away)
    from paper_1702_06813_amd import rendermap
    monkeypatch.setenv("RM_LOG", "1")
    slot = 64 * 32 * 8

    def sized(schedule):
        ctx = rm.Context(0)
        monkeypatch.setitem(rendermap._ctxs, 0, ctx)
        ctx.set_tile(64, 32)
        ctx.set_bin_cap(64)
        ctx.set_bin_pool(0)
        ctx.set_schedule(schedule)
        capfd.readouterr()
        out = rm.align_cost_grad(mesh, scan, T, EPS)
        return ctx, out, _slots(capfd)

    _, ref, (asked, _, need) = sized(0)
    ctx, whole, (_, _, need1) = sized(1)
    assert torch.equal(whole, ref)
    # (scratch grows to a quarter more than it needs, at least 1 MiB)
    left = max(need1 + need1 // 4, 1 << 20) - (need - 4096 * slot)
    assert 0 < left // slot < asked
    ctx.set_schedule(0)
    out = torch.empty_like(ref)
    with rm.Graph(torch.device("cuda", 0)) as g:
        rm.align_cost_grad(mesh, scan, T, EPS, out=out)
    for _ in range(3):
        out.fill_(float("nan"))
        g.replay()
        assert torch.equal(out, ref)
    torch.cuda.synchronize()
    del g
