"""Calls whose blocks do not all start together: results and the workspace's next
calls are those of an ordinary call, however late a block starts and however
short the wait for it is."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch

    from paper_2112_10034_amd import cox

    cox.lib()
    return torch, cox


def same(torch, a, b):
    return all(torch.equal(u.view(torch.uint8), v.view(torch.uint8)) for u, v in zip(a, b))


# (schedule, chunks): two blocks; a ragged last chunk; more chunks than the 256
# lanes of the final tree; several chunks a block and a combine of blocks below
# and above 256 threads
SHAPES = [((4, 4, 0), 2), ((1, 1, 0), 37), ((4, 4, 0), 300), ((8, 32, 64), 700), ((2, 2, 5), 91)]


@pytest.mark.parametrize("polls", [0, 3, 512])
@pytest.mark.parametrize("cfg,nch", SHAPES)
@pytest.mark.parametrize("dtype,acc,dot", [("int32", 0, False), ("float32", 0, False), ("bfloat16", 1, False),
                                           ("float32", 1, True), ("bfloat16", 0, True)])
def test_reduce_with_a_late_block(dev, dtype, acc, dot, cfg, nch, polls):
    torch, cox = dev
    S = 32 * cfg[0] * cfg[1]
    n = nch * S - S // 3
    g = torch.Generator(device="cuda").manual_seed(nch + polls)

    def draw():
        if dtype == "int32":
            return torch.randint(-1 << 20, 1 << 20, (n,), dtype=torch.int32, device="cuda", generator=g)
        return torch.randn(n, device="cuda", generator=g).to(getattr(torch, dtype))

    def ordinary(x, y):
        return cox.warp_reduce(x, acc, cfg=cfg) if y is None else cox.warp_dot(x, y, acc, cfg=cfg)

    blocks = min(nch, cfg[2] or 1 << 30)
    ws = cox.workspace(cox.OP_DOT if dot else cox.OP_REDUCE, cox._CODES[getattr(torch, dtype)], n, cfg=cfg)
    for away in sorted({0, blocks // 2, blocks - 1}):
        x1, x2 = draw(), draw()
        y1, y2 = (draw(), draw()) if dot else (None, None)
        want1, want2 = ordinary(x1, y1), ordinary(x2, y2)
        got = cox.warp_reduce_away(x1, y1, acc, cfg, away, polls)
        after = ordinary(x2, y2)
        assert same(torch, got, want1), away
        assert same(torch, after, want2), away
        ws.status()


def test_refuses_a_negative_block(dev):
    torch, cox = dev
    x = torch.ones(4096, dtype=torch.int32, device="cuda")
    for kw in ({"away_block": -1}, {"polls": 513}):
        with pytest.raises(cox.CoxError) as e:
            cox.warp_reduce_away(x, **kw)
        assert e.value.code == 1


# the three kernels for short inputs: two chunks, a ragged last one, as many
# chunks as the block has threads and one more, the most chunks
SHORT = [("scan", 8193), ("scan", 65613), ("scan", 1 << 18), ("scan", (1 << 18) + 1), ("scan", 512 * 8192),
         ("scan", 512 * 8192 + 5), ("scan", 1 << 23), ("compact", 8193), ("compact", 100001), ("compact", 513 * 8192),
         ("compact", (1 << 23) + 1), ("compact", 1 << 24)]


@pytest.mark.parametrize("polls", [0, 3, 512])
@pytest.mark.parametrize("what,n", SHORT)
def test_short_scan_and_compaction_with_a_late_block(dev, what, n, polls):
    torch, cox = dev
    g = torch.Generator(device="cuda").manual_seed(n)
    chunk = 16384 if n > 1 << 23 else 8192
    blocks = -(-n // chunk)

    def draw():
        return torch.randint(-1 << 20, 1 << 20, (n,), dtype=torch.int32, device="cuda", generator=g)

    def want(x):
        return torch.cumsum(x, 0, dtype=torch.int32) if what == "scan" else x[x > 0]

    def check(r, w, away):
        if what == "compact":
            assert int(r[1]) == w.numel(), away
            r = r[0][:w.numel()]
        assert torch.equal(r, w), away

    ordinary = cox.warp_scan if what == "scan" else cox.ballot_compact
    late = cox.warp_scan_away if what == "scan" else cox.ballot_compact_away
    ws = cox.workspace(cox.OP_SCAN if what == "scan" else cox.OP_COMPACT, cox.I32, n)
    for away in sorted({0, blocks // 2, blocks - 1}):
        x1, x2 = draw(), draw()
        w1, w2 = want(x1), want(x2)
        got = late(x1, away, polls)
        after = ordinary(x2)
        check(got, w1, away)
        check(after, w2, away)
        ws.status()


def test_longer_inputs_are_refused(dev):
    torch, cox = dev
    x = torch.ones((1 << 24) + 1, dtype=torch.int32, device="cuda")
    for call in (cox.warp_scan_away, cox.ballot_compact_away):
        with pytest.raises(cox.CoxError) as e:
            call(x)
        assert e.value.code == 6
