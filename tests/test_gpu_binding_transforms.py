"""Calls on tensors that have no data of their own (inside vmap, grad and
forward-mode transforms, fake tensors) raise, from the native module as from the
Python code."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch

    from paper_2112_10034_amd import cox

    cox.lib()
    return torch, cox


def calls(torch, cox):
    off = torch.tensor([0, 32, 64], device="cuda")
    yield "i", cox.warp_scan
    yield "i", lambda x: cox.ballot_compact(x)[0]
    yield "i", cox.tile_sort
    yield "i", lambda x: cox.tile_reduce(x, 4)
    yield "i", lambda x: cox.warp_masked(x, 512)[0]
    yield "i", lambda x: cox.warp_reduce_blocks_i32(x)[0]
    yield "i", lambda x: cox.segmented(x, off, 2)[1]
    yield "f", lambda x: cox.warp_reduce(x)[0]
    yield "f", lambda x: cox.warp_dot(x, x)[0]
    yield "b", cox.integral_image


def test_transforms_raise(dev):
    torch, cox = dev
    f = torch.arange(256, device="cuda", dtype=torch.float32)
    tensors = {"f": f.view(4, 64), "i": f.int().view(4, 64), "b": f.to(torch.uint8).view(4, 8, 8)}
    for kind, call in calls(torch, cox):
        x = tensors[kind]
        call(x[0].contiguous())  # the workspace is there
        with pytest.raises(RuntimeError):
            torch.func.vmap(call)(x)
        if kind == "f":
            with pytest.raises(RuntimeError):
                torch.func.grad(lambda v: call(v)[0])(x[0])
            with pytest.raises(RuntimeError):
                torch.func.jvp(call, (x[0],), (x[0],))
        call(x[0].contiguous())  # and calls work as before


def test_fake_tensors_raise(dev):
    torch, cox = dev
    from torch._subclasses.fake_tensor import FakeTensorMode

    x = torch.arange(64, dtype=torch.int32, device="cuda")
    cox.warp_scan(x)
    with FakeTensorMode() as mode:
        with pytest.raises(Exception):
            cox.warp_scan(mode.from_tensor(x))
    assert int(cox.warp_scan(x)[-1]) == 2016
