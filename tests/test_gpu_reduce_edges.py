"""Reductions where the kernel's paths meet: one chunk alone, the partial last
chunk cut inside a vector (every remainder), fewer elements than one vector,
grids on both sides of the grouped done count, and every schedule width of
the final combine, bit for bit against the oracle."""
import numpy as np
import pytest

from paper_2112_10034_amd import inputs

pytestmark = pytest.mark.gpu


def bf16(f):
    return inputs._to_bf16_bits(f)


def up(a):
    import torch

    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(a).cuda()


def data(dtype, n, seed):
    xi, _, f = inputs.primitive_inputs(n, seed=seed)
    return {"i32": xi, "f32": f, "bf16": bf16(f)}[dtype]


def check(oracle_mod, cox, dtype, n, cfg, acc, dot):
    x = data(dtype, n, n + 1)
    y = data(dtype, n, n + 2) if dot else None
    code = {"i32": cox.I32, "f32": cox.F32, "bf16": cox.BF16}[dtype]
    k, W = cfg[:2] if cfg else cox.default_cfg(cox.OP_DOT if dot else cox.OP_REDUCE, code)[:2]
    if dot:
        op, ot = oracle_mod.dot(x, y, k, W, acc)
        t, p = cox.warp_dot(up(x), up(y), acc, cfg=cfg)
    else:
        op, ot = oracle_mod.reduce(x, k, W, acc) if dtype != "i32" else oracle_mod.reduce(x, k, W)
        t, p = cox.warp_reduce(up(x), acc, cfg=cfg)
    what = (dtype, n, cfg, acc, dot)
    assert p.cpu().numpy().tobytes() == np.ascontiguousarray(op).tobytes(), what
    if dtype == "i32":
        assert int(t.cpu()[0]) == ot, what
    else:
        assert t.cpu().numpy().view(np.uint64)[0] == np.float64(ot).view(np.uint64), what


@pytest.mark.parametrize("dtype", ["i32", "f32", "bf16"])
@pytest.mark.parametrize("acc", [0, 1])
@pytest.mark.parametrize("dot", [False, True])
def test_edges(oracle_mod, dtype, acc, dot):
    from paper_2112_10034_amd import cox

    if dtype == "i32" and (acc or dot):
        pytest.skip("not offered")
    for n in [1, 2, 3, 5, 7, 8, 9, 15, 31, 33]:
        check(oracle_mod, cox, dtype, n, (16, 1), acc, dot)
    for r in range(9):  # one full chunk and a cut second one
        check(oracle_mod, cox, dtype, 4096 + 1024 + r, (16, 8), acc, dot)
    check(oracle_mod, cox, dtype, 4096, (16, 8), acc, dot)
    check(oracle_mod, cox, dtype, 4096, (16, 8, 3), acc, dot)
    for n in (300, 32 * 64 - 1, 32 * 65, 32 * 66 + 1, 32 * 300 + 17):  # one-warp chunks: up to 301 blocks
        check(oracle_mod, cox, dtype, n, (1, 1), acc, dot)
        check(oracle_mod, cox, dtype, n, (2, 2, 66), acc, dot)
    for W in (1, 2, 4, 8, 16, 32):
        check(oracle_mod, cox, dtype, 100003, (8, W), acc, dot)
    for n in (1000, 65613, 1000003):
        check(oracle_mod, cox, dtype, n, None, acc, dot)
