"""The log-sRGB tone map of the loss over its whole range: with a = 1, m = 0
and no specular shading the render is Ld, and against a black observation a
single point's loss is the squared map, its albedo gradient 2 Gamma Gamma' Ld.
Compared with extended precision from 1e-30 to the largest float, on both sides
of the map's join (log(1 + x) = 0.0031308), at zero, below it, at infinity and
for NaN.  Tolerance: the map is good to a few units in the last place of a
double (1e-15, twice that when squared; 1e-14 asserted), the gradient is
rounded to single precision (6e-8; 2e-7 asserted)."""
import numpy as np
import pytest
import torch

from paper_2304_05669_amd import fipt

pytestmark = pytest.mark.gpu
SIG = (0.1, 0.5)


def _loss(x, masked):
    sh = torch.zeros((15, 1), device="cuda")
    sh[0] = x
    mat = torch.tensor([[1.0], [1.0], [1.0], [0.3], [0.0]], device="cuda")
    obs = torch.zeros((3, 1), device="cuda")
    if masked:
        buf, g, _, _ = fipt.fipt_render_loss_masked(sh, mat, obs, SIG, None, 0.0, fipt.TONEMAP_LOG_SRGB)
    else:
        buf, g, _ = fipt.fipt_render_loss(sh, mat, obs, SIG, fipt.TONEMAP_LOG_SRGB)
    return buf[0].item(), g[0, 0].item()


def _map(x):
    x = np.longdouble(x)
    u = np.log1p(x)
    if u <= np.longdouble(0.0031308):
        return 12.92 * u, 12.92 / (1 + x)
    p = u ** (np.longdouble(1) / np.longdouble(2.4))
    return (np.longdouble(1.055) * p - np.longdouble(0.055),
            np.longdouble(1.055 / 2.4) * p / (u * (1 + x)))


def _values():
    rng = np.random.default_rng(4)
    join = np.expm1(0.0031308)
    v = np.concatenate([10.0 ** rng.uniform(-30, 38, 40), 10.0 ** rng.uniform(-4, 2, 60),
                        join * (1 + np.array([-1e-3, -1e-6, 1e-6, 1e-3])),
                        [1.0, 0.41421356, 0.41421360, 3.0, 3.4028235e38, 1e-38]])
    return [float(np.float32(x)) for x in v]


@pytest.mark.parametrize("masked", [False, True])
def test_log_srgb_map_and_derivative(masked):
    for x in _values():
        val, der = _map(x)
        loss, grad = _loss(x, masked)
        assert abs(loss - float(val * val)) <= 1e-14 * float(val * val), x
        want = float(2 * val * der * np.longdouble(x))
        if want > 1e-37:
            assert abs(grad - want) <= 2e-7 * want, x


def test_log_srgb_map_outside_its_range():
    for x in (0.0, -1.0, -3e38, float("nan")):
        assert _loss(x, False)[0] == 0.0
    assert _loss(float("inf"), False)[0] == float("inf")
