"""The hand-out of points to the wavefronts of the persistent bake and
refinement kernels: at launch sizes around the number of wavefronts (one
point each, shares one short or one over, points left to the counters), every
point is baked, and to the bits of the same point in a larger launch (the
random numbers of a point are those of its index)."""
import pytest
import torch

import synth
from paper_2304_05669_amd import fipt

pytestmark = pytest.mark.gpu
SIG = (0.1, 0.5)


@pytest.fixture(scope="module")
def tiny_points_gpu():
    sc = synth.tiny_box()
    sc.cameras[0].width = sc.cameras[0].height = 128      # 16,384 points
    scene = fipt.Scene(sc.verts, sc.tris, device=0)
    scene.set_radiance(torch.from_numpy(sc.cache).cuda(), fipt.CACHE_TRIANGLE,
                       torch.from_numpy(sc.emission).cuda())
    planes, tri = fipt.fipt_gen_points(scene, sc.cameras)
    yield scene, planes, tri
    torch.cuda.synchronize()
    scene.destroy()


def _head(t, n):
    return t[..., :n].contiguous()


SIZES = [1, 7, 8, 9, 4095, 4096, 4097, 5119, 5120, 5121, 5129, 10241]


def test_bake_every_point_at_any_launch_size(tiny_points_gpu):
    scene, planes, tri = tiny_points_gpu
    full = fipt.fipt_bake(scene, planes, tri, 6, 3, SIG, 11)
    for n in SIZES:
        out = torch.full((3 + 6 * len(SIG), n), float("nan"), device="cuda")
        for _ in range(2):      # a second launch on the next counter slot
            fipt.fipt_bake(scene, _head(planes, n), _head(tri, n), 6, 3, SIG, 11, out=out)
        assert torch.equal(out, _head(full, n)), n


def test_refine_every_point_at_any_launch_size(tiny_points_gpu):
    scene, planes, tri = tiny_points_gpu
    grid = torch.rand((5, 4, 4, 4), generator=torch.Generator().manual_seed(3)).cuda()
    box = ([0.0] * 3, [1.0] * 3)
    full = fipt.fipt_refine(scene, planes, tri, 6, 3, SIG, 11, grid, *box)
    for n in SIZES:
        out = torch.full((3 + 6 * len(SIG), n), float("nan"), device="cuda")
        fipt.fipt_refine(scene, _head(planes, n), _head(tri, n), 6, 3, SIG, 11, grid, *box, out=out)
        assert torch.equal(out, _head(full, n)), n
