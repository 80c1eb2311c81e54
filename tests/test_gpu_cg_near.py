"""Conjugate gradient when no block reads outside its window (the blocks
exchange tagged words instead of meeting at barriers): chunk counts around
one, 16, 32 and 256, last chunks shorter than a halo, every compiled
schedule, back-to-back solves on one workspace (which holds the earlier
solve's words), a far solve between near ones, and early ends."""
import numpy as np
import pytest

from paper_2112_10034_amd import inputs

pytestmark = pytest.mark.gpu


def solve(sysm, x0, it, tol, cfg):
    import torch

    from paper_2112_10034_amd import cox

    x = torch.from_numpy(x0.copy()).cuda()
    res, hist = cox.cg_solve(*(torch.from_numpy(a).cuda() for a in sysm), x, it, tol, cfg=cfg)
    cox.workspace(cox.OP_CG, cox.F32, x0.size, cfg=cfg).status()
    k, reason = (int(v) for v in res.cpu())
    return x.cpu().numpy(), k, reason, hist.cpu().numpy()[: k + 1]


def check(oracle_mod, sysm, it, tol, cfg, x0=None):
    n = sysm[3].size
    x0 = np.zeros(n, np.float32) if x0 is None else x0
    print("cg near", n, cfg, it, flush=True)
    got = solve(sysm, x0, it, tol, cfg)
    want = oracle_mod.cg(*sysm, x0, it, tol, *cfg[:2])
    assert got[1:3] == tuple(want[1:3])
    assert got[0].tobytes() == want[0].tobytes() and got[3].tobytes() == want[3].tobytes()


@pytest.mark.parametrize("R", [1, 2, 4, 8])
@pytest.mark.parametrize("W", [8, 16, 32])
def test_every_schedule(oracle_mod, R, W):
    S = 32 * W * R
    for nch, tail in ((1, 0), (2, 1), (3, 63), (16, 65), (17, 0)):
        check(oracle_mod, inputs.cg_tridiag((nch - 1) * S + (tail or S), seed=nch), 9, 0.0, (R, W))


@pytest.mark.parametrize("nch,tail", [(15, 5), (16, 200), (17, 1), (31, 64), (32, 256), (33, 2), (64, 100), (65, 256),
                                      (255, 10), (256, 256), (256, 3)])
def test_chunk_counts(oracle_mod, nch, tail):
    check(oracle_mod, inputs.cg_tridiag((nch - 1) * 256 + tail, seed=nch + tail), 12, 0.0, (1, 8))


def test_solves_in_a_row_and_early_ends(oracle_mod):
    near = inputs.cg_tridiag(40 * 256 + 7, seed=3)
    other = inputs.cg_tridiag(5 * 4096 + 11, seed=4)
    far = inputs.cg_irregular(9000, seed=5)
    for _ in range(2):
        check(oracle_mod, near, 15, 0.0, (1, 8))
        check(oracle_mod, near, 15, 0.0, (1, 8), x0=np.linspace(-1, 1, near[3].size).astype(np.float32))
        check(oracle_mod, far, 10, 0.0, (4, 32))
        check(oracle_mod, other, 20, 0.0, (4, 32))
    check(oracle_mod, near, 400, 1e-5, (1, 8))  # converges
    check(oracle_mod, near, 0, 0.0, (1, 8))
    n = 600  # <p, A p> is not positive in the second chunk's rows
    indef = (np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32),
             np.where(np.arange(n) < 300, 1, -1).astype(np.float32), np.ones(n, np.float32))
    check(oracle_mod, indef, 10, 0.0, (1, 8))
