"""The hash-grid forward pass's scratch: inference asks for no more than the
encoding it writes (64 floats per point of a run), any scratch of at least one
point's encoding gives the bits of the kernel that needs none, and without
memory that kernel runs."""
import pytest
import torch

from paper_2304_05669_amd import fipt
from test_gpu_hashgrid_encode import HI, LO, _params, _plain, _points

pytestmark = pytest.mark.gpu


def test_inference_takes_the_encoding_and_no_more():
    n = 300001
    params, pos = _params(), _points(n, 3)
    out = torch.empty((5, n), device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    fipt.fipt_hashgrid_forward(params, pos, LO, HI, out=out)
    torch.cuda.synchronize()
    took = torch.cuda.max_memory_allocated() - before
    assert took <= 64 * 4 * n + (1 << 20), took
    assert torch.cuda.memory_allocated() == before


@pytest.mark.parametrize("n,floats", [(1, 64), (5, 64), (300, 64 * 65 + 63), (1000, 64 * 256), (1000, 64 * 4000)])
def test_any_scratch_gives_the_same_bits(n, floats):
    params, pos = _params(), _points(n, n)
    out = torch.full((5, n), float("nan"), device="cuda")
    scratch = torch.full((floats + 64,), 7.0, device="cuda")

    def call(size):
        return fipt.lib().fipt_hashgrid_forward_scratch(
            params.data_ptr(), pos.data_ptr(), n, n, fipt._f32_array(LO, 3), fipt._f32_array(HI, 3), out.data_ptr(),
            n, scratch.data_ptr(), size, fipt._stream())

    assert call(floats) == 0
    assert torch.equal(out, _plain(params, pos))
    assert (scratch[floats:] == 7.0).all()
    assert call(63) == fipt.EINVAL


def test_without_memory(monkeypatch):
    params, pos = _params(), _points(1000, 9)

    def no_memory(n, device):
        raise torch.cuda.OutOfMemoryError("no memory")

    monkeypatch.setattr(fipt, "hashgrid_scratch", no_memory)
    assert torch.equal(fipt.fipt_hashgrid_forward(params, pos, LO, HI), _plain(params, pos))


@pytest.mark.parametrize("groups", [(3, 4, 0), (3, 4, 1), (3, 1, 0), (3, 1, 1)])
def test_forms_agree_where_they_change(groups):
    """At the sizes between which one kernel does the whole pass: a multiple of
    the CUs in workgroups of 256 points, and a point more."""
    num, den, more = groups
    n = 256 * num * torch.cuda.get_device_properties(0).multi_processor_count // den + more
    params, pos = _params(), _points(n, 4)
    assert torch.equal(fipt.fipt_hashgrid_forward(params, pos, LO, HI), _plain(params, pos))
