"""The work that programs hand to this library, as measured cases.

A case is one call (or one plan replay, or one solve) through the public
Python entry points of ``paper_2112_10034_amd.cox``, on inputs that are
already on the GPU, with the distributions the library's own workloads have
(``paper_2112_10034_amd/inputs.py`` states them; here they are drawn on the
GPU so that full sizes take milliseconds).  ``listed()`` names one case per
part of the primitive set, from the smallest calls to the full sizes that
the benchmark runs; ``draw()`` spreads the same calls over their sizes,
types and options, odd sizes included.
"""
import math

import torch

from paper_2112_10034_amd import cox, inputs

_ACC = {"plain": cox.PLAIN, "twosum": cox.TWOSUM}
_DTYPE = {"i32": torch.int32, "f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # per-block sums and per-warp positive counts of one batch: the
        # smallest of the library's own workloads, bound by the call itself
        {"name": "block_reduce_2p20", "kind": "block_reduce", "n": 1 << 20},
        # the sum of a small, ragged vector: a few chunks, one of them
        # partial; what a program pays for one small reduction
        {"name": "sum_f32_65613", "kind": "reduce", "op": "sum", "dtype": "f32", "acc": "plain", "n": 65613},
        # the compensated dot product over two full-size bfloat16 vectors,
        # the precision workload's most arithmetic per byte
        {"name": "dot_bf16_twosum_2p28", "kind": "reduce", "op": "dot", "dtype": "bf16", "acc": "twosum",
         "n": 1 << 28},
        # an ordinary prefix sum, of a length that is a multiple of nothing
        {"name": "scan_1000003", "kind": "scan", "n": 1000003},
        # stable compaction of a full-size batch, about half of it kept
        {"name": "compact_2p28", "kind": "compact", "n": 1 << 28},
        # 32-key group sort of an ordinary batch with a partial last group
        {"name": "sort32_4194321", "kind": "sort", "tile": 32, "n": (1 << 22) + 17},
        # groups wider than a wave
        {"name": "sort1024_2p26", "kind": "sort", "tile": 1024, "n": 1 << 26},
        # shuffles and votes under partial masks, half the lanes in them
        {"name": "masked_d512_2p26", "kind": "masked", "density": 512, "n": 1 << 26},
        # 10,000 uneven float segments, all three results, replayed from the
        # plan that a serving loop keeps
        {"name": "plan_f32_10000", "kind": "segmented", "plan": True, "dtype": "f32", "nseg": 10000},
        # a few hundred integer segments in one direct call
        {"name": "segmented_i32_300", "kind": "segmented", "plan": False, "dtype": "i32", "nseg": 300},
        # summed-area table of a large image
        {"name": "image_8192x8192", "kind": "image", "height": 8192, "width": 8192},
        # 50 iterations of conjugate gradient on a system that fits on chip
        {"name": "cg_2p20_50", "kind": "cg", "n": 1 << 20, "iterations": 50},
    ]


def _log_size(rng, lo, hi):
    """A whole number between lo and hi, spread over the logarithm; one in
    four is a power of two."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.25:
        n = 1 << max(0, round(math.log2(n)))
    return max(lo, min(hi, n))


def draw(rng):
    kind = rng.choice(["block_reduce", "reduce", "reduce", "scan", "compact", "sort", "sort", "masked", "segmented",
                       "segmented", "image", "cg"])
    if kind == "block_reduce":
        return {"kind": kind, "n": _log_size(rng, 1 << 8, 1 << 24)}
    if kind == "reduce":
        op = rng.choice(["sum", "dot"])
        dtype = rng.choice(["f32", "bf16"] if op == "dot" else ["i32", "f32", "bf16"])
        acc = "plain" if dtype == "i32" else rng.choice(["plain", "twosum"])
        return {"kind": kind, "op": op, "dtype": dtype, "acc": acc, "n": _log_size(rng, 1 << 10, 1 << 27)}
    if kind in ("scan", "compact"):
        return {"kind": kind, "n": _log_size(rng, 1 << 10, 1 << 27)}
    if kind == "sort":
        return {"kind": kind, "tile": rng.choice([32, 32, 64, 128, 256, 512, 1024]), "n": _log_size(rng, 1 << 10, 1 << 26)}
    if kind == "masked":
        # whole warps, as the call wants
        return {"kind": kind, "density": rng.choice(list(inputs.MASK_DENSITIES)),
                "n": 32 * _log_size(rng, 1 << 5, 1 << 21)}
    if kind == "segmented":
        return {"kind": kind, "plan": rng.random() < 0.5, "dtype": rng.choice(["i32", "f32"]),
                "nseg": _log_size(rng, 10, 9000)}
    if kind == "image":
        return {"kind": kind, "height": _log_size(rng, 64, 6000), "width": _log_size(rng, 64, 6000)}
    return {"kind": kind, "n": _log_size(rng, 1 << 10, 1 << 20), "iterations": rng.randint(10, 50)}


# ------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _ints(g, n, lo, hi):
    """int32 uniform in [lo, hi]"""
    return torch.randint(lo, hi + 1, (n,), dtype=torch.int32, device="cuda", generator=g)


def _bits(g, n):
    """uint32 uniform, carried in int32"""
    return torch.randint(-(1 << 31), 1 << 31, (n,), dtype=torch.int32, device="cuda", generator=g)


def _precision(g, n, dtype):
    """magnitudes 10^U(-3, 3), random signs"""
    out = torch.empty(n, dtype=dtype, device="cuda")
    for a in range(0, n, 1 << 26):
        m = min(n - a, 1 << 26)
        v = torch.rand(m, device="cuda", generator=g).mul_(6.0).sub_(3.0)
        v = torch.pow(10.0, v)
        s = torch.randint(0, 2, (m,), dtype=torch.int8, device="cuda", generator=g)
        out[a:a + m] = torch.where(s == 0, v, -v).to(dtype)
    return out


def _reduce_input(g, case):
    n, dtype = case["n"], _DTYPE[case["dtype"]]
    if dtype == torch.int32:
        return _ints(g, n, -(1 << 20), 1 << 20)
    if case["acc"] == "twosum":
        return _precision(g, n, dtype)
    return torch.randn(n, device="cuda", generator=g).to(dtype)


def _offsets(case, seed):
    """CSR offsets: the workload's lengths in an order of the seed's own"""
    lens = torch.from_numpy(inputs.segment_offsets(nseg=case["nseg"])).diff()
    order = torch.randperm(lens.numel(), generator=torch.Generator().manual_seed(seed))
    return torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(lens[order], 0)])


def _tridiagonal(g, n):
    """(off-diagonal [n - 1], diagonal [n], right-hand side [n])"""
    off = -torch.rand(max(n - 1, 0), device="cuda", generator=g)
    dia = 3.0 + torch.rand(n, device="cuda", generator=g)
    rhs = torch.rand(n, device="cuda", generator=g) * 2.0 - 1.0
    return off, dia, rhs


def _csr(off, dia):
    n = dia.numel()
    i = torch.arange(n, dtype=torch.int32, device="cuda")
    cols = torch.stack([i - 1, i, i + 1], dim=1)
    vals = torch.zeros(n, 3, device="cuda")
    vals[1:, 0] = off
    vals[:, 1] = dia
    vals[:-1, 2] = off
    valid = (cols >= 0) & (cols < n)
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(valid.sum(dim=1), 0).to(torch.int32)
    return rp, cols[valid].contiguous(), vals[valid].contiguous()


def prepare(case, seed):
    kind, g = case["kind"], _gen(seed)
    s = {"kind": kind}
    if kind == "block_reduce":
        s["x"] = _ints(g, case["n"], -1000, 1000)
    elif kind == "reduce":
        s["acc"] = _ACC[case["acc"]]
        s["x"] = _reduce_input(g, case)
        s["y"] = _reduce_input(g, case) if case["op"] == "dot" else None
    elif kind in ("scan", "compact"):
        s["x"] = _ints(g, case["n"], -(1 << 20), 1 << 20)
        if kind == "compact":
            # a buffer of the call's capacity, kept: what lies past the kept
            # elements is the caller's
            s["out"] = torch.zeros_like(s["x"])
    elif kind == "sort":
        s["tile"] = case["tile"]
        s["x"] = _bits(g, case["n"])
    elif kind == "masked":
        s["density"] = case["density"]
        s["x"] = _ints(g, case["n"], -(1 << 20), 1 << 20)
    elif kind == "segmented":
        off = _offsets(case, seed)
        total = int(off[-1])
        x = _ints(g, total, -(1 << 20), 1 << 20) if case["dtype"] == "i32" else \
            torch.randn(total, device="cuda", generator=g)
        s["x"], s["off"] = x, off.cuda()
        # the default schedule (a tuned one may differ from run to run, and
        # with it the rounding of float results)
        s["plan"] = cox.Plan(x, s["off"], autotune=False) if case["plan"] else None
    elif kind == "image":
        s["img"] = torch.randint(0, 256, (case["height"], case["width"]), dtype=torch.uint8, device="cuda",
                                 generator=g)
    else:
        off, dia, rhs = _tridiagonal(g, case["n"])
        s["csr"], s["b"] = _csr(off, dia), rhs
        s["x"] = torch.zeros_like(rhs)
        s["iterations"] = case["iterations"]
    return s


def run(s):
    kind = s["kind"]
    if kind == "block_reduce":
        return cox.warp_reduce_blocks_i32(s["x"])
    if kind == "reduce":
        if s["y"] is None:
            return cox.warp_reduce(s["x"], s["acc"])
        return cox.warp_dot(s["x"], s["y"], s["acc"])
    if kind == "scan":
        return cox.warp_scan(s["x"])
    if kind == "compact":
        return cox.ballot_compact(s["x"], out=s["out"])
    if kind == "sort":
        return cox.tile_sort(s["x"], s["tile"])
    if kind == "masked":
        return cox.warp_masked(s["x"], s["density"])
    if kind == "segmented":
        if s["plan"] is not None:
            return s["plan"].execute()
        return cox.segmented(s["x"], s["off"])
    if kind == "image":
        return cox.integral_image(s["img"])
    # every solve starts from zero
    x = s["x"].zero_()
    result, history = cox.cg_solve(*s["csr"], s["b"], x, s["iterations"])
    return x, result, history


def work(case):
    kind = case["kind"]
    if kind == "block_reduce":
        n = case["n"]
        return {"bytes": 4 * n + 4 * -(-n // 256) + 4 * -(-n // 32), "flops": n}
    if kind == "reduce":
        n, arrays = case["n"], 2 if case["op"] == "dot" else 1
        per = {"plain": 1, "twosum": 7}[case["acc"]] if arrays == 1 else {"plain": 2, "twosum": 11}[case["acc"]]
        return {"bytes": n * arrays * (2 if case["dtype"] == "bf16" else 4) + 8, "flops": per * n}
    if kind == "scan":
        return {"bytes": 8 * case["n"], "flops": case["n"]}
    if kind == "compact":
        return {"bytes": 6 * case["n"] + 8, "flops": case["n"]}  # half of the elements are kept
    if kind == "sort":
        t = int(math.log2(case["tile"]))
        return {"bytes": 8 * case["n"], "flops": case["n"] * t * (t + 1) // 4}  # comparators of the network
    if kind == "masked":
        return {"bytes": 8 * case["n"] + case["n"] // 2, "flops": case["n"]}
    if kind == "segmented":
        nseg, n = case["nseg"], int(inputs.segment_offsets(nseg=case["nseg"])[-1])
        return {"bytes": 10 * n + 24 * nseg, "flops": 2 * n}
    if kind == "image":
        p = case["height"] * case["width"]
        return {"bytes": 5 * p, "flops": 2 * p}
    n, it = case["n"], case["iterations"]
    return {"bytes": 4 * (n + 1) + 24 * n + 12 * n + 8 * (it + 1), "flops": it * 16 * n}


# -------------------------------------------------------------------- exact
def _sum64(x, y=None):
    tot = torch.zeros((), dtype=torch.float64, device="cuda")
    for a in range(0, x.numel(), 1 << 26):
        v = x[a:a + (1 << 26)].double()
        tot += (v if y is None else v * y[a:a + (1 << 26)].double()).sum()
    return tot.reshape(1)


def _exact_segments(x, off):
    """totals, restarting scan and compaction of float segments in 64 bits"""
    n, dev = x.numel(), x.device
    lens = off[1:] - off[:-1]
    seg = torch.repeat_interleave(torch.arange(lens.numel(), device=dev), lens)
    cum = torch.cat([torch.zeros(1, dtype=torch.float64, device=dev), torch.cumsum(x.double(), 0)])
    totals = cum[off[1:]] - cum[off[:-1]]
    scan = cum[1:] - cum[off[:-1]][seg]
    keep = x > 0
    kc = torch.cat([torch.zeros(1, dtype=torch.int64, device=dev), torch.cumsum(keep.long(), 0)])
    where = off[:-1][seg] + kc[:-1] - kc[off[:-1]][seg]
    out = torch.zeros(n, dtype=torch.float64, device=dev)
    out[where[keep]] = x[keep].double()
    return totals, scan, out, kc[off[1:]] - kc[off[:-1]]


def _exact_cg(off, dia, b, iterations):
    off, dia, b = off.double(), dia.double(), b.double()

    def mul(v):
        y = dia * v
        y[1:] += off * v[:-1]
        y[:-1] += off * v[1:]
        return y

    x, r, p = torch.zeros_like(b), b.clone(), b.clone()
    rr = [(r * r).sum()]
    for _ in range(iterations):
        q = mul(p)
        alpha = rr[-1] / (p * q).sum()
        x = x + alpha * p
        r = r - alpha * q
        rr.append((r * r).sum())
        p = r + (rr[-1] / rr[-2]) * p
    result = torch.tensor([iterations, cox.CG_MAX_ITER], dtype=torch.int32)
    return x, result, torch.stack(rr)


def exact(case, seed):
    """The floating-point results in 64 bits.  Whole-number results have one
    right value, which every version of the library gives."""
    kind, g = case["kind"], _gen(seed)
    if kind == "reduce" and case["dtype"] != "i32":
        x = _reduce_input(g, case)
        y = _reduce_input(g, case) if case["op"] == "dot" else None
        if case["acc"] == "twosum":
            return _sum64(x, y), None  # a compensated chunk's two words have no value of their own
        op = cox.OP_DOT if y is not None else cox.OP_REDUCE
        k, W, _ = cox.default_cfg(op, {"f32": cox.F32, "bf16": cox.BF16}[case["dtype"]])
        S = 32 * k * W
        parts = [_sum64(x[a:a + S], None if y is None else y[a:a + S]) for a in range(0, x.numel(), S)]
        return _sum64(x, y), torch.cat(parts)
    if kind == "segmented" and case["dtype"] == "f32":
        off = _offsets(case, seed).cuda()
        return _exact_segments(torch.randn(int(off[-1]), device="cuda", generator=g), off)
    if kind == "cg":
        return _exact_cg(*_tridiagonal(g, case["n"]), case["iterations"])
    return None
