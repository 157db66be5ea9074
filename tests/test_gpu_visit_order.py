"""Which of two triangles a bake reports where a ray meets both within the last
bit of the distance, about one ray in 10^10.  The order of visits decides it,
so that order is part of the result: children of equal entry distance keep
their places in the node step's sorting network, in the bake as in the ray cast
and the refinement.

The three values are of points at which an order by distance and reference
reported the other triangle: (seed, point, plane, value) of a bake of a small
room with a radiance of its own for every triangle, which moves such a value by
a whole radiance over the 256 samples (1.4e-3 to 3.4e-3).  The rounding of 256
single-precision additions is at most 256 2^-24, 1.6e-5 of a value below 1."""
import numpy as np
import pytest
import torch

import synth
from paper_2304_05669_amd import fipt

pytestmark = pytest.mark.gpu

SPP = 256
NEAR_TIES = [(4, 293538, 12, 0.869845331), (11, 548763, 14, 0.832255781), (16, 440221, 6, 0.487023592)]


def test_near_ties_keep_the_distance_order():
    sc = synth.serving_rooms(seed=0, n_cams=8, which=[0])[0]
    radiance = np.random.Generator(np.random.PCG64(1)).integers(0, 256, size=(3, sc.n_tris)) / 128.0
    radiance = torch.from_numpy(radiance.astype(np.float32)).cuda()
    scene = fipt.Scene(sc.verts, sc.tris, device=0)
    try:
        scene.set_radiance(radiance, fipt.CACHE_TRIANGLE, torch.zeros_like(radiance))
        planes, tri = fipt.fipt_gen_points(scene, sc.cameras)
        for seed, point, plane, want in NEAR_TIES:
            got = fipt.fipt_bake(scene, planes, tri, SPP, SPP, sc.sigma, seed)
            assert abs(float(got[plane, point]) - want) <= SPP * 2.0 ** -24, (seed, point)
    finally:
        scene.destroy()
