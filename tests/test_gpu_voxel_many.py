"""More voxels of many pixels than the pooling launch has wavefronts: 40,000 (a
wavefront takes two), and 67.2 million, with which a launch of one wavefront
each would exceed the 2^32 threads of a HIP launch (no error: voxels were left
unwritten).  Nine pixels per voxel whose values are 0 to 8 plus the channel: the
mean is 4 plus the channel, exactly."""
import numpy as np
import pytest
import torch

from paper_2304_05669_amd import fipt

pytestmark = pytest.mark.gpu

PER = 9


@pytest.mark.parametrize("R,filled", [(64, 40_000), (512, 67_200_000)])
def test_every_voxel_of_many_pixels(R, filled):
    n = PER * filled
    assert R == 64 or filled * 64 > 2 ** 32
    v = torch.arange(filled, device="cuda").repeat_interleave(PER)
    pos = torch.empty((3, n), device="cuda")
    for k, div in enumerate((1, R, R * R)):
        pos[k] = (torch.div(v, div, rounding_mode="floor") % R + 0.5) / R
    pos_host = pos.cpu().numpy()
    del v, pos
    obs = torch.empty((3, n), device="cuda")
    obs.view(3, filled, PER)[:] = torch.arange(float(PER), device="cuda")
    obs += torch.arange(3.0, device="cuda")[:, None]
    plan = fipt.VoxelPlan(pos_host, R, np.zeros(3), np.ones(3))
    del pos_host
    out = torch.full((3, R ** 3), float("nan"), device="cuda")
    plan.pool(obs, out=out)
    torch.cuda.synchronize()
    for c in range(3):
        assert (out[c, :filled] == 4.0 + c).all()
        assert not out[c, filled:].any()
