"""The fused loss's grid adjoint over work units of few and many columns: one
point in each of the first n cells of one brick of nodes makes one unit of n
columns (two units above 256), at the edges of its wavefronts.  Against the
adjoint that sums the points itself, of the fused call's own per-point
gradients: a column's sum is one product rounded to single precision, and each
side rounds a node's total, so they differ by at most three roundings of
the sum of magnitudes."""
import numpy as np
import pytest
import torch

import synth
from paper_2304_05669_amd import fipt
from test_gpu_loss import DEV, SIG, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 192, 193, 255, 256, 257, 343])
def test_units_of_every_width(n):
    R = 8
    rng = np.random.default_rng(n)
    cell = np.arange(343)[:n]
    pos = np.stack([cell % 7, cell // 7 % 7, cell // 49]) + rng.uniform(0.1, 0.9, size=(3, n))
    pos = (pos / (R - 1)).astype(np.float32)
    plan = fipt.GridPlan(pos, R, np.zeros(3, np.float32), np.ones(3, np.float32))
    grid = _t(synth.material_grid(R, seed=3))
    sh_q, obs_q = (plan.permute(_t(a)) for a in (synth.random_shading(n, 6, seed=n),
                                                  synth.random_observations(n, seed=n + 1)))
    gq = torch.empty((5, n), device=DEV)
    _, got = plan.render_loss(grid, sh_q, obs_q, SIG, 0, grad_points=gq)
    gp = torch.empty_like(gq)
    gp[:, torch.from_numpy(plan.order()).to(DEV).long()] = gq
    want, magnitude = plan.scatter(gp), plan.scatter(gp.abs())
    err = (got.double() - want.double()).abs().reshape(5, -1)
    assert float(want.abs().max()) > 0
    assert (err <= 3 * 2.0 ** -24 * 1.001 * magnitude.double().reshape(5, -1)).all()
