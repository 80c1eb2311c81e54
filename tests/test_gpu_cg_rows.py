"""Conjugate gradient without far columns on rows of differing length: empty
rows, rows within and beyond the entries that a thread holds in registers,
columns up to the halo's edge on both sides, zeros of either sign in b and x,
and a last chunk with few rows."""
import numpy as np
import pytest

from test_gpu_cg_near import check

pytestmark = pytest.mark.gpu


def banded(n, most, seed):
    """a symmetric system with up to most off-diagonal entries per row, none
    farther than 64 rows away, and some rows and columns without any entry"""
    g = np.random.default_rng(seed)
    off = g.choice([1, 2, 5, 17, 63, 64], size=most // 2, replace=False) if most else np.zeros(0, np.int64)
    i = np.concatenate([np.arange(n - d) for d in off if d < n] or [np.zeros(0, np.int64)])
    j = np.concatenate([np.arange(d, n) for d in off if d < n] or [np.zeros(0, np.int64)])
    empty = g.random(n) < 0.02
    keep = (g.random(i.size) < 0.7) & ~empty[i] & ~empty[j]
    i, j = i[keep], j[keep]
    v = -g.random(i.size, dtype=np.float32)
    k = np.flatnonzero(~empty)
    rows, cols = np.concatenate([i, j, k]), np.concatenate([j, i, k])
    vals = np.concatenate([v, v, np.float32(most + 1) + g.random(k.size, dtype=np.float32)])
    order = np.lexsort((g.random(rows.size), rows))  # entries of a row in any order
    rp = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(rows, minlength=n), out=rp[1:])
    b = g.random(n, dtype=np.float32) * np.float32(2) - np.float32(1)
    b[empty | (g.random(n) < 0.05)] = 0.0
    b[g.random(n) < 0.02] = -0.0
    b[empty] = 0.0
    return rp, cols[order].astype(np.int32), vals[order], b


@pytest.mark.parametrize("most", [0, 2, 4, 6, 10])
@pytest.mark.parametrize("cfg", [(1, 8), (2, 16), (4, 32), (8, 8)])
def test_rows(oracle_mod, cfg, most):
    S = 32 * cfg[0] * cfg[1]
    for nch, tail in ((1, S // 2 + 1), (2, 3), (5, 70), (6, S)):
        n = (nch - 1) * S + tail
        x0 = np.where(np.arange(n) % 3 == 0, np.float32(-0.0), np.float32(0.25))
        check(oracle_mod, banded(n, most, nch + most), 8, 0.0, cfg, x0=x0.astype(np.float32))
