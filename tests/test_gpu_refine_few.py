"""The refinement's form for few points (at most 12 per CU) and the one for
more give the same bits: the points of a launch one above the line, and the same
points in launches at the line and below it; and as the chunked form above 10
roughness levels is untouched by the line, it agrees across it as well."""
import pytest
import torch

import synth
from paper_2304_05669_amd import fipt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [6, 11])
def test_forms_agree_across_the_line(levels):
    line = 12 * torch.cuda.get_device_properties(0).multi_processor_count
    sc = synth.serving_rooms(seed=0, n_cams=1, which=[0])[0]
    scene = fipt.Scene(sc.verts, sc.tris, device=0)
    try:
        em = torch.from_numpy(sc.emission).cuda()
        rad = torch.rand((3, sc.n_tris), generator=torch.Generator().manual_seed(1)).cuda()
        scene.set_radiance(rad, fipt.CACHE_TRIANGLE, em)
        planes, tri = fipt.fipt_gen_points(scene, sc.cameras)
        sigma = [0.05 + 0.9 * i / levels for i in range(levels)]
        grid = torch.rand((5, 8, 8, 8), generator=torch.Generator().manual_seed(2)).cuda()
        box = (sc.bmin.tolist(), sc.bmax.tolist())
        first = (planes.shape[1] - line - 1) // 2

        def refine(n):
            return fipt.fipt_refine(scene, planes[:, first:first + n].contiguous(), tri[first:first + n].contiguous(),
                                    8, 8, sigma, 7, grid, *box)

        above = refine(line + 1)
        assert float(above.abs().max()) > 0
        for n in (line, line - 1, 65):
            assert torch.equal(refine(n), above[:, :n].contiguous()), n
    finally:
        scene.destroy()
