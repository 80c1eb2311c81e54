"""Scans and compactions of short inputs (default schedule: one chunk per
block, every block reading all earlier aggregates at once) at the edges of
their chunks and of the sizes at which the chunk grows, on a workspace used
again by the other sizes and by the look-back kernel."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

def sizes():
    out = [1, 3, 4, 255, 256, 257, 8191, 8192, 8193, 65613, 1000003]
    for v in (1 << 18, 1 << 22, 1 << 23, 1 << 24):
        out += [v - 1, v, v + 1]
    return out


def test_short_scan_and_compaction():
    import torch

    from paper_2112_10034_amd import cox

    rng = np.random.default_rng(5)
    for n in sizes() + sizes()[:12]:
        x = rng.integers(-(1 << 31), 1 << 31, size=n, dtype=np.int64).astype(np.int32)
        xg = torch.from_numpy(x).cuda()
        print("short", n, flush=True)
        want = np.cumsum(x.astype(np.int64)).astype(np.int32)  # wraps as the additions do
        assert np.array_equal(cox.warp_scan(xg).cpu().numpy(), want), n
        assert np.array_equal(cox.warp_scan_noalloc(xg).cpu().numpy(), want), n
        out = torch.full((n + 8,), 77, dtype=torch.int32, device="cuda")
        for shift in (0, 3):  # an output that starts off a 16-byte boundary too
            got, cnt = cox.ballot_compact(xg, out=out[shift:shift + n])
            keep = x[x > 0]
            assert int(cnt.cpu()[0]) == keep.size, n
            assert np.array_equal(got.cpu().numpy()[:keep.size], keep), (n, shift)
            assert int(out[shift + n]) == 77
    cox.workspace(cox.OP_SCAN, cox.I32, 1).status()


@pytest.mark.parametrize("n", [1000, 65613, 1000003])
def test_short_calls_keep_what_was_accepted(n):
    """A workspace of the look-back kernel's size and an output that is the
    input are still taken, with the same results."""
    import torch

    from paper_2112_10034_amd import cox

    L = cox.lib()
    k, W, _ = cox.default_cfg(cox.OP_SCAN)
    x = torch.randint(-1000, 1000, (n,), dtype=torch.int32, device="cuda")
    want = torch.cumsum(x.long(), 0).to(torch.int32)
    ws = cox.Workspace(256 + 128 * (-(-n // (32 * k * W)) + 1))
    y = torch.empty_like(x)
    for _ in range(2):
        code = L.cox_warp_scan(C.c_void_p(x.data_ptr()), C.c_void_p(y.data_ptr()), n, None,
                               C.c_void_p(ws.tensor.data_ptr()), ws.nbytes, None)
        torch.cuda.synchronize()
        assert code == 0 and torch.equal(y, want)
    keep = x[x > 0]
    z = x.clone()
    _, cnt = cox.ballot_compact(z, out=z)
    assert int(cnt.cpu()[0]) == keep.numel() and torch.equal(z[:keep.numel()], keep)


def test_short_calls_in_a_graph():
    """Replays of a captured scan and compaction, with eager calls on other
    buffers between them."""
    import torch

    from paper_2112_10034_amd import cox

    n = 300007
    x = torch.randint(-1000, 1000, (n,), dtype=torch.int32, device="cuda")
    y, out = torch.empty_like(x), torch.empty_like(x)
    cnt = torch.empty(1, dtype=torch.int64, device="cuda")
    cox.warp_scan(x, out=y), cox.ballot_compact(x, out=out, count=cnt)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(3):
            cox.warp_scan(x, out=y)
            cox.ballot_compact(x, out=out, count=cnt)
    for r in range(4):
        x.copy_(torch.randint(-1000, 1000, (n,), dtype=torch.int32, device="cuda"))
        g.replay()
        assert torch.equal(y, torch.cumsum(x.long(), 0).to(torch.int32)), r
        keep = x[x > 0]
        assert int(cnt.cpu()[0]) == keep.numel() and torch.equal(out[:keep.numel()], keep), r
        z = torch.ones(5000 + r, dtype=torch.int32, device="cuda")
        assert int(cox.warp_scan(z)[-1]) == 5000 + r
