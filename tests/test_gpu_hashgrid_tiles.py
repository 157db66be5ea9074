"""The hash-grid backward pass around its 64-point tiles: one point, one tile
and one more, workgroups that take a single tile and ones that take two
(40,001 points: more than 512 tiles), against the oracle; the gradients of all
levels and weights, twice the same bits, and untouched entries exactly zero.
Tolerance as for the backward parity at 20,000 points: single-precision sums
of the same products."""
import numpy as np
import pytest
import torch

from oracle import hashgrid as hg
from paper_2304_05669_amd import fipt
from test_gpu_hashgrid import HI, LO, _close, _params, _points, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 64, 65, 40001])
def test_backward_tiles(n):
    params, x = _params(5), _points(n, 6)
    gy = np.random.default_rng(7).standard_normal((5, n)).astype(np.float32)
    P, X, G = _t(params), _t(x), _t(gy)
    plan = fipt.HashGridPlan(X, LO, HI)
    ws = torch.full((int(fipt.lib().fipt_hashgrid_workspace_floats(n)),), float("nan"), device="cuda")
    g1 = fipt.fipt_hashgrid_backward(plan, P, G, workspace=ws)
    g2 = fipt.fipt_hashgrid_backward(plan, P, G)
    assert torch.equal(g1, g2)
    want = hg.backward(params, x, LO, HI, gy)
    a = g1.cpu().numpy()
    ends = np.cumsum([hg.N_TABLE, hg.N_W1, hg.N_W2, hg.N_W3])
    for k, name in enumerate(("W1", "W2", "W3")):
        _close(a[ends[k]:ends[k + 1]], want[ends[k]:ends[k + 1]], 1e-3, name)
    for lv in range(hg.LEVELS):
        sl = slice(lv * hg.T * hg.FEATURES, (lv + 1) * hg.T * hg.FEATURES)
        _close(a[sl], want[sl], 1e-3, f"table level {lv}")
    untouched = want[:hg.N_TABLE] == 0
    assert np.all(a[:hg.N_TABLE][untouched] == 0.0)
