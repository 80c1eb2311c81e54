"""The binding's native path and its Python path give the same results, keep
the caller's outputs, and raise the same errors; a cached workspace that is
too small is replaced."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch

    from paper_2112_10034_amd import cox

    cox.lib()
    return torch, cox


class Declining:
    """A native module that declines every call: the Python path runs."""

    def __getattr__(self, name):
        return lambda *a: None


def calls(torch, cox, n):
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randint(-1000, 1000, (n,), dtype=torch.int32, device="cuda", generator=g)
    f = torch.randn(n, device="cuda", generator=g)
    h = f.to(torch.bfloat16)
    m = x[: n // 32 * 32]
    off = torch.tensor([0, n // 3, n // 3, n], dtype=torch.int64, device="cuda")
    img = (x[: n // 32 * 32].reshape(32, -1) & 255).to(torch.uint8)
    buf = torch.zeros_like(x)
    yield "blocks", lambda: cox.warp_reduce_blocks_i32(x)
    for v in (x, f, h):
        yield f"sum {v.dtype}", lambda v=v: cox.warp_reduce(v)
        yield f"sum no partials {v.dtype}", lambda v=v: cox.warp_reduce(v, partials=False)[:1]
    for v in (f, h):
        yield f"sum twosum {v.dtype}", lambda v=v: cox.warp_reduce(v, cox.TWOSUM)
        yield f"dot {v.dtype}", lambda v=v: cox.warp_dot(v, v, cox.TWOSUM)
    yield "scan", lambda: cox.warp_scan(x)
    yield "compact", lambda: cox.ballot_compact(x, out=buf.zero_())
    for t in (32, 64, 1024):
        yield f"sort {t}", lambda t=t: cox.tile_sort(x, t)
    yield "tile", lambda: cox.tile_reduce(x, 8)
    yield "masked", lambda: cox.warp_masked(m, 512)
    for v in (x, f):
        yield f"segmented {v.dtype}", lambda v=v: cox.segmented(v, off)
        yield f"segmented scan {v.dtype}", lambda v=v: cox.segmented(v, off, cox.SEG_SCAN)[1]
    yield "image", lambda: cox.integral_image(img)


def flat(r):
    return [v.clone() for v in r] if isinstance(r, (tuple, list)) else [r.clone()]


@pytest.mark.parametrize("n", [32, 1023, 70001])
def test_native_and_python_paths_agree(dev, monkeypatch, n):
    torch, cox = dev
    for what, call in calls(torch, cox, n):
        call()  # the workspace is there
        a = flat(call())
        with monkeypatch.context() as m:
            m.setattr(cox, "_native", Declining())
            b = flat(call())
        assert len(a) == len(b), what
        for u, v in zip(a, b):
            assert u.shape == v.shape and u.dtype == v.dtype and u.device == v.device, what
            assert torch.equal(u.view(torch.uint8), v.view(torch.uint8)), what


def test_outputs_given_by_the_caller(dev):
    torch, cox = dev
    x = torch.arange(1, 4097, dtype=torch.int32, device="cuda")
    cox.warp_scan(x)
    y = torch.empty_like(x)
    assert cox.warp_scan(x, out=y) is y
    s, w = torch.empty(16, dtype=torch.int32, device="cuda"), torch.empty(128, dtype=torch.int32, device="cuda")
    r = cox.warp_reduce_blocks_i32(x, s, w)
    assert r[0] is s and r[1] is w
    k = x.flip(0).contiguous()
    assert cox.tile_sort(k, out=k) is k
    tot, part = cox.warp_reduce(x, partials=False)
    assert part is None and int(tot) == 4096 * 4097 // 2
    st, yy, oc, c = cox.segmented(x, torch.tensor([0, 4096], device="cuda"), cox.SEG_REDUCE)
    assert yy is None and oc is None and c is None and int(st) == 4096 * 4097 // 2


def test_refused_calls_stay_refused(dev):
    torch, cox = dev
    x = torch.arange(4096, dtype=torch.int32, device="cuda")
    cox.warp_scan(x), cox.ballot_compact(x), cox.warp_reduce(x)
    cox.warp_dot(x.float(), x.float())
    for bad in (x.cpu(), x.float(), [1, 2], None):
        for fn in (cox.warp_scan, cox.ballot_compact, cox.tile_sort, cox.warp_reduce_blocks_i32):
            with pytest.raises((TypeError, AttributeError)):
                fn(bad)
    with pytest.raises(ValueError):
        cox.warp_scan(x.reshape(64, 64).t())
    with pytest.raises(ValueError):
        cox.warp_dot(x.float(), x[:5].float())
    with pytest.raises(TypeError):
        cox.warp_dot(x.float(), x)
    with pytest.raises(TypeError):
        cox.tile_reduce(x, 4.0)
    for code, call in ((3, lambda: cox.warp_scan(x[1:])), (3, lambda: cox.tile_sort(x[1:])),
                       (1, lambda: cox.tile_sort(x, 48)), (2, lambda: cox.warp_reduce(x, cox.TWOSUM)),
                       (2, lambda: cox.warp_dot(x, x)), (1, lambda: cox.warp_masked(x, 2000)),
                       (1, lambda: cox.warp_masked(x[:33].clone(), 5)), (1, lambda: cox.tile_reduce(x, 3))):
        with pytest.raises(cox.CoxError) as e:
            call()
        assert e.value.code == code


def test_a_small_workspace_grows(dev):
    torch, cox = dev
    saved = dict(cox._ws_cache)
    try:
        cox._ws_cache.clear()
        small = torch.ones(1000, dtype=torch.int32, device="cuda")
        big = torch.ones((1 << 24) + 5, dtype=torch.int32, device="cuda")
        for x in (small, big, small, big):
            assert int(cox.warp_scan(x)[-1]) == x.numel()
            assert int(cox.warp_reduce(x)[0]) == x.numel()
            assert int(cox.ballot_compact(x)[1]) == x.numel()
    finally:
        cox._ws_cache.update(saved)


def test_current_stream_is_used(dev):
    torch, cox = dev
    x = torch.ones(1 << 20, dtype=torch.int32, device="cuda")
    cox.warp_scan(x)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        assert cox._stream() == s.cuda_stream
        y = x + 1
        z = cox.warp_scan(y)
    s.synchronize()
    assert int(z[-1]) == 2 << 20
