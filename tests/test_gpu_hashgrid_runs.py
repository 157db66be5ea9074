"""The weight gradients of the hash-grid backward pass where many small
contributions follow a few large ones: a single-precision sum over too many
points loses them whole.

Every value is a power of two, so the sums are known: all points at the box's
first corner with tables of ones (the encoding is 1), W1 and W2 such that both
hidden layers are 1, W3 of +1 and -1 in turn such that every output is 1/2, and
an output gradient that is 1 for the first 32,768 points (64 for each of 512
workgroups, were a workgroup's points 64 of every 32,768) and 2^-21 after.
Beside 64 contributions of 1/4 those of 2^-23 are below half a unit in the
last place, four together too.  In runs of at most 2,048 points at most one run
holds both kinds, so at most 2,048 x 2^-23 is lost, with the result's own
rounding; in one sum over each workgroup's 8,192 points it is 0.496 of 8192.5."""
import numpy as np
import pytest
import torch

from oracle import hashgrid as hg
from paper_2304_05669_amd import fipt

pytestmark = pytest.mark.gpu

LO, HI = (0.0, 0.0, 0.0), (1.0, 1.0, 1.0)
N, FIRST = 1 << 22, 1 << 15


def test_small_contributions_survive_large_ones():
    ends = np.cumsum([hg.N_TABLE, hg.N_W1, hg.N_W2, hg.N_W3])
    params = torch.zeros((fipt.HG_PARAMS,), device="cuda")
    params[:ends[0]] = 1.0
    params[ends[0]:ends[1]].view(64, 64)[:, 0] = 1.0
    params[ends[1]:ends[2]].view(64, 64).fill_diagonal_(1.0)
    sign = 1.0 - 2.0 * (torch.arange(64, device="cuda") % 2)
    params[ends[2]:ends[3]].view(5, 64)[:] = sign
    plan = fipt.HashGridPlan(torch.zeros((3, N), device="cuda"), LO, HI)
    gy = torch.zeros((5, N), device="cuda")
    gy[0, :FIRST] = 1.0
    gy[0, FIRST:] = 2.0 ** -21
    g = fipt.fipt_hashgrid_backward(plan, params, gy).cpu().numpy().astype(np.float64)
    total = 0.25 * (FIRST + (N - FIRST) * 2.0 ** -21)      # of d3 = gy y (1 - y)
    tol = 2048 * 2.0 ** -23 + total * 2.0 ** -23
    sign = sign.cpu().numpy()
    w1, w2 = g[ends[0]:ends[1]].reshape(64, 64), g[ends[1]:ends[2]].reshape(64, 64)
    w3 = g[ends[2]:ends[3]].reshape(5, 64)
    np.testing.assert_allclose(w3[0], total, rtol=0, atol=tol)
    np.testing.assert_allclose(w2, np.outer(sign, np.full(64, total)), rtol=0, atol=tol)
    np.testing.assert_allclose(w1, np.outer(sign, np.full(64, total)), rtol=0, atol=tol)
    assert not w3[1:].any()
