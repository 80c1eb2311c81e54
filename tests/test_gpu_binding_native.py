"""The binding's native module makes the ordinary calls, and leaves numbers
that are no C ints to the Python code, as ctypes takes them."""
import pytest

from tests.test_gpu_binding import calls

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch

    from paper_2112_10034_amd import cox

    cox.lib()
    return torch, cox


class Recorder:
    def __init__(self, native):
        self.native, self.answers = native, []

    def __getattr__(self, name):
        fn = getattr(self.native, name)

        def call(*args):
            r = fn(*args)
            self.answers.append((name, r))
            return r

        return call


@pytest.mark.parametrize("n", [1023, 70001])
def test_the_native_module_answers(dev, monkeypatch, n):
    torch, cox = dev
    for what, call in calls(torch, cox, n):
        call()  # the workspace is there
        rec = Recorder(cox._native)
        with monkeypatch.context() as m:
            m.setattr(cox, "_native", rec)
            call()
        assert len(rec.answers) == 1, what
        name, r = rec.answers[0]
        assert r is not None and type(r) is not int, (what, name, r)


def test_numbers_past_a_c_int(dev):
    torch, cox = dev
    x = torch.randint(-100, 100, (4096,), dtype=torch.int32, device="cuda")
    assert torch.equal(cox.tile_sort(x, (1 << 64) + 32), cox.tile_sort(x, 32))
    assert torch.equal(cox.tile_sort(x, (1 << 32) + 64), cox.tile_sort(x, 64))
    for u, v in zip(cox.warp_masked(x, (1 << 70) + 512), cox.warp_masked(x, 512)):
        assert torch.equal(u, v)
    off = torch.tensor([0, 4096], device="cuda")
    cox.segmented(x, off)
    a = cox.segmented(x, off, (1 << 64) + 1)
    assert int(a[0]) == int(x.sum()) and a[1] is None
    for bad in (1 << 62, (1 << 63) - 1, 1 << 63, 1 << 90):
        with pytest.raises(cox.CoxError):
            cox.tile_reduce(x, bad)
        with pytest.raises(cox.CoxError):
            cox.tile_sort(x, bad + 1)
        with pytest.raises(cox.CoxError):
            cox.warp_masked(x, bad * 4 - 1)


def test_an_output_selection_that_is_no_int(dev):
    torch, cox = dev
    x = torch.arange(4096, dtype=torch.int32, device="cuda")
    off = torch.tensor([0, 4096], device="cuda")
    cox.segmented(x, off)
    for which in (2.0, "2", None):
        with pytest.raises(TypeError):
            cox.segmented(x, off, which)
    assert cox.segmented(x, off, True)[1] is None
