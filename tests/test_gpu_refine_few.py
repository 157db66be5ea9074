"""The refinement at three wavefronts per SIMD and at four gives the same bits:
launches on both sides of each size at which the form changes (12 points per CU,
17, 24, 33 and 36), against the same points of the largest launch; for the
per-lane paths and for the chunked form above 10 roughness levels."""
import pytest
import torch

import synth
from paper_2304_05669_amd import fipt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [6, 11])
def test_forms_agree_across_the_lines(levels):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    lines = [12 * cus, 17 * cus, 24 * cus, 33 * cus, 36 * cus]
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
        first = (planes.shape[1] - lines[-1] - 1) // 2

        def refine(n):
            return fipt.fipt_refine(scene, planes[:, first:first + n].contiguous(), tri[first:first + n].contiguous(),
                                    4, 4, sigma, 7, grid, *box)

        full = refine(lines[-1] + 1)
        assert float(full.abs().max()) > 0
        for n in [65] + [k + more for k in lines for more in (0, 1)]:
            assert torch.equal(refine(n), full[:, :n].contiguous()), n
    finally:
        scene.destroy()
