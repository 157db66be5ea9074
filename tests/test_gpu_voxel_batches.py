"""The voxel pooling's batches and the two forms of the occupancy words, at
their edges: voxels of 0 to 4 pixels (one batch of four), 5 to 8 (one of eight) and
more (a wavefront each, 256 staged at a time), against the oracle bit for bit;
and grids of a multiple of four voxels per axis read with 16-byte loads
against the same grid at an address that takes the general form, which the
oracle tests cover.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import cache as oc
from paper_2304_05669_amd import fipt

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("R", [3, 8])
def test_pool_batches_bitwise(R):
    rng = np.random.default_rng(R)
    counts = np.resize([0, 1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 0, 63, 64, 65, 255, 256, 257, 513], R ** 3)
    vox = rng.permutation(np.repeat(np.arange(R ** 3), counts))
    ijk = np.stack([vox % R, vox // R % R, vox // (R * R)])
    x = ((ijk + 0.5) / R).astype(np.float32)
    obs = rng.uniform(0, 5, size=x.shape).astype(np.float32)
    lo, hi = np.zeros(3, np.float32), np.ones(3, np.float32)
    out = torch.full((3, R ** 3), float("nan"), device=DEV)
    fipt.VoxelPlan(x, R, lo, hi).pool(torch.from_numpy(obs).to(DEV), out=out)
    got = out.cpu().numpy()
    want, n = oc.voxel_pool(x, obs, lo, hi, R)
    assert np.array_equal(np.asarray(n).ravel(), counts)
    np.testing.assert_array_equal(got, want.astype(np.float32))


# 1, 8, 27 and 125 bricks: a wavefront takes four
@pytest.mark.parametrize("R", [4, 8, 12, 20])
def test_word_forms_agree(R):
    sc = synth.tiny_box()
    tris = np.asarray(sc.tris)
    scene = fipt.Scene(sc.verts, sc.tris, 0)
    planes, tri = fipt.fipt_gen_points(scene, sc.cameras)
    em = torch.from_numpy(sc.emission).to(DEV)
    rng = np.random.default_rng(R)
    n = R ** 3
    c = rng.uniform(0.5, 2.0, size=(3, n)).astype(np.float32)
    c[:, rng.uniform(size=n) < 0.5] = 0.0               # empty voxels
    c[rng.integers(0, 3, size=n // 2), rng.integers(0, n, size=n // 2)] = 0.0   # single channels
    buf = torch.zeros(3 * n + 8, device=DEV)
    got = []
    for off in (0, 1):                                  # 16-byte aligned, and not
        cache = buf[off:off + 3 * n].view(3, n)
        cache.copy_(torch.from_numpy(c))
        assert (cache.data_ptr() % 16 == 0) == (off == 0)
        scene.set_voxel_radiance(cache, R, sc.bmin.tolist(), sc.bmax.tolist(), em)
        got.append(fipt.fipt_bake(scene, planes, tri, 8, 4, sc.sigma, 3))
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1])
    assert float(got[0].abs().max()) > 0 and tris.shape[0] > 0
