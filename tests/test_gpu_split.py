"""Records cut into slices (calls with few, full tiles) against the same call
with one workgroup per record, which cuts none: bit-identical records and
images, also where bins overflow into regions or into the every-cluster path."""
import numpy as np
import pytest

from gpu_helpers import EPS, oracle_map, workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap,pool", [(0, -1), (256, 0), (256, 1 << 20)])
@pytest.mark.parametrize("tile", [(64, 32), (32, 32), (16, 16)])
@pytest.mark.parametrize("n_poses", [1, 5])
def test_slices_against_whole_records(n_poses, tile, cap, pool):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1702_06813_amd as rm
    w = workload("kinect")
    mesh = rm.Mesh.from_arrays(*oracle_map("kinect")).prepare()
    scan = rm.scan_image(torch.from_numpy(w.scan_depth).cuda(), cam=w.cam)
    T = torch.from_numpy(np.ascontiguousarray(w.poses[:n_poses].reshape(-1, 12))).cuda()
    vn = torch.nn.functional.normalize(torch.randn(mesh.xyz.shape, generator=torch.Generator().manual_seed(3))).cuda()
    ctx = rm.context()
    got = {}
    ctx.set_tile(*tile)
    ctx.set_bin_cap(cap)
    ctx.set_bin_pool(pool)
    try:
        for schedule in (1, 0, 0):                 # the second pass of the split call on used scratch
            ctx.set_schedule(schedule)
            r = rm.render_depth(mesh, w.cam, T)
            now = [rm.align_cost(mesh, scan, T, EPS), rm.align_cost_grad(mesh, scan, T, EPS),
                   rm.icp_cost_grad(mesh, scan, T, vn), r["tri"], r["cls"], r["depth"].view(torch.int32)]
            for k, x in enumerate(now):
                if schedule == 1:
                    got[k] = x.clone()
                else:
                    assert torch.equal(x, got[k]), k
    finally:
        ctx.set_schedule(0)
        ctx.set_tile(0, 0)
        ctx.set_bin_cap(0)
        ctx.set_bin_pool(-1)
