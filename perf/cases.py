"""The work this library is measured on: plain calls, ragged batches, row
tables, row softmax and the NLL loss, through the Python entry points that a
program calls, with the context, offsets and output buffers that it keeps.

A case is a dict of plain values; `listed()` names the fixed ones, `draw(rng)`
gives another of the same ranges, `prepare` makes a program's state from a seed,
`run` makes one pass, `work` says what the pass cannot do without and `exact`
gives its outputs in 64 bits with plain torch.
"""
import math

import numpy as np
import torch

from paper_2207_00257_amd import api

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
SIZE = {"f32": 4, "bf16": 2, "f16": 2}
# the dtype pairs of the rows of a mixed row table, as a serving batch mixes its requests
MIX = (("f32", "f32"), ("bf16", "bf16"), ("f32", "f32"), ("f16", "f32"), ("f32", "bf16"))
MOST_ELEMS = 1 << 28  # elements of the largest case
F16_ROW = 1 << 13  # longest row whose quotients float16 holds without subnormals


def listed():
    return [
        # the smallest calls: a short vector, launch latency and the host side
        dict(name="plain_f32_1000", op="plain", n=1000, in_dt="f32", out_dt="f32", accum="f32", in_off=0, out_off=0),
        # the small plain configuration (2^20 binary32), resident in the caches
        dict(name="plain_f32_2p20", op="plain", n=1 << 20, in_dt="f32", out_dt="f32", accum="f32", in_off=0, out_off=0),
        # an ordinary long serving request: bfloat16 in and out, a length that is no multiple of anything
        dict(name="plain_bf16_5000011", op="plain", n=5000011, in_dt="bf16", out_dt="bf16", accum="f32", in_off=0,
             out_off=0),
        # the precision configuration: 2^26 bfloat16 of wide range, compensated sum, binary32 out
        dict(name="plain_bf16_2p26_kahan", op="plain", n=1 << 26, in_dt="bf16", out_dt="f32", accum="kahan", in_off=0,
             out_off=0),
        # the bandwidth configuration: 2^28 binary32
        dict(name="plain_f32_2p28", op="plain", n=1 << 28, in_dt="f32", out_dt="f32", accum="f32", in_off=0, out_off=0),
        # a small ragged batch: what a batched call costs before its bytes do
        dict(name="csr_64_small", op="csr", rows=64, lo=32, hi=4096, in_dt="f32", out_dt="f32", accum="f32"),
        # the ragged configuration: 4096 rows, lengths log-uniform in [32, 2^20]
        dict(name="csr_4096", op="csr", rows=4096, lo=32, hi=1 << 20, in_dt="f32", out_dt="f32", accum="f32"),
        # many equal short rows (the short-rows benchmark)
        dict(name="csr_2p20x256", op="csr", rows=1 << 20, lo=256, hi=256, in_dt="f32", out_dt="f32", accum="f32"),
        # many rows of mixed short and middling lengths (the same benchmark's ragged leg)
        dict(name="csr_200000", op="csr", rows=200000, lo=1, hi=4096, in_dt="f32", out_dt="f32", accum="f32"),
        # a serving group: a row table of mixed dtypes, lengths of the request trace
        dict(name="rows_16_mixed", op="rows", rows=16, lo=1 << 8, hi=1 << 24, accum="f32"),
        # row softmax with log-sum-exp over the ragged configuration's rows
        dict(name="softmax_4096", op="softmax", rows=4096, lo=32, hi=1 << 20),
        # the NLL loss of a batch of class log-probabilities (mean, weights, ignored samples)
        dict(name="nll_2p20x1000", op="nll", n=1 << 20, c=1000, reduction="mean", weight=True, accum="f32"),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def _lengths_range(rng, rows, hi_max, most):
    """(lo, hi) of the lengths of `rows` rows, at most about `most` elements together."""
    hi = _log_uniform(rng, 16, hi_max)
    lo = hi if rng.random() < 0.25 else _log_uniform(rng, 1, hi)

    def mean(lo, hi):
        return float(lo) if hi <= lo else (hi - lo) / math.log(hi / lo)

    while rows * mean(lo, hi) > most and hi > 16:
        hi = max(16, hi // 2)
        lo = min(lo, hi)
    return lo, hi


def draw(rng):
    op = rng.choice(["plain"] * 5 + ["csr"] * 4 + ["rows", "softmax", "nll"])
    dts = [rng.choice(["f32", "f32", "bf16", "f16"]) for _ in range(2)]
    if rng.random() < 0.6:
        dts[1] = dts[0]
    accum = "kahan" if rng.random() < 0.25 else "f32"
    # outputs sum to one over a row: float16 holds them for short rows only
    if op == "plain":
        # views into a larger array: starts that are no line's, alike or not in input and output
        in_off = rng.randrange(1, 64) if rng.random() < 0.3 else 0
        out_off = in_off if rng.random() < 0.7 else rng.randrange(0, 64)
        n = _log_uniform(rng, 1 << 8, 1 << 27)
        out_dt = "f32" if dts[1] == "f16" and n > F16_ROW else dts[1]
        return dict(op=op, n=n, in_dt=dts[0], out_dt=out_dt, accum=accum, in_off=in_off, out_off=out_off)
    if op == "csr":
        rows = _log_uniform(rng, 1, 1 << 20)
        lo, hi = _lengths_range(rng, rows, 1 << 22, MOST_ELEMS // 2)
        out_dt = "f32" if dts[1] == "f16" and hi > F16_ROW else dts[1]
        return dict(op=op, rows=rows, lo=lo, hi=hi, in_dt=dts[0], out_dt=out_dt, accum=accum)
    if op == "rows":
        rows = _log_uniform(rng, 4, 64)
        lo, hi = _lengths_range(rng, rows, 1 << 24, MOST_ELEMS // 4)
        return dict(op=op, rows=rows, lo=lo, hi=hi, accum=accum)
    if op == "softmax":
        rows = _log_uniform(rng, 1, 1 << 20)
        lo, hi = _lengths_range(rng, rows, 1 << 21, MOST_ELEMS // 2)
        return dict(op=op, rows=rows, lo=lo, hi=hi)
    return dict(op=op, n=_log_uniform(rng, 1 << 10, 1 << 20), c=_log_uniform(rng, 10, 1000),
                reduction=rng.choice(["mean", "mean", "sum", "none"]), weight=rng.random() < 0.5, accum=accum)


# ---- inputs ------------------------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _lengths(case):
    """The case's row lengths, log-uniform in [lo, hi]: the same for every seed, so that its outputs have one shape."""
    rng = np.random.Generator(np.random.PCG64([case["rows"], case["lo"], case["hi"]]))
    lo, hi = case["lo"], case["hi"]
    u = rng.random(case["rows"])
    return np.clip(np.floor(np.exp(np.log(lo) + u * (np.log(hi + 1.0) - np.log(lo)))), lo, hi).astype(np.int64)


def _offsets(case, seed):
    """CSR offsets: the case's lengths in an order of the seed's."""
    order = np.random.Generator(np.random.PCG64(int(seed))).permutation(case["rows"])
    offs = np.zeros(case["rows"] + 1, np.int64)
    np.cumsum(_lengths(case)[order], out=offs[1:])
    return offs


def _uniform(n, seed):
    """U[0.5, 1.5), the plain workloads' values."""
    return torch.rand(n, device="cuda", generator=_gen(seed)).add_(0.5)


def _lognormal(n, seed, sigma):
    return torch.empty(n, device="cuda").normal_(0.0, sigma, generator=_gen(seed)).exp_()


def _plain_input(case, seed):
    # wide-range values for the compensated sum, the plain workload's otherwise
    n = case["n"]
    wide = case["accum"] == "kahan" and case["in_dt"] != "f16"
    return (_lognormal(n, seed, 2.0) if wide else _uniform(n, seed)).to(DTYPES[case["in_dt"]])


def _row_input(k, n, seed):
    return _uniform(n, seed * 1009 + k).to(DTYPES[MIX[k % len(MIX)][0]])


def _nll_inputs(case, seed):
    n, c = case["n"], case["c"]
    g = _gen(seed)
    logp = torch.empty(n, c, device="cuda").exponential_(1.0 / 3.0, generator=g).neg_()
    target = torch.randint(0, c, (n,), device="cuda", generator=g)
    target[torch.rand(n, device="cuda", generator=g) < 0.05] = -100
    weight = torch.rand(c, device="cuda", generator=g).add_(0.5) if case["weight"] else None
    return logp, target, weight


def _view(buffer_dtype, off, n):
    return torch.empty(off + n, dtype=buffer_dtype, device="cuda")[off:]


def prepare(case, seed):
    op = case["op"]
    state = dict(case=case, ctx=api.Context())
    if op == "plain":
        inp = _view(DTYPES[case["in_dt"]], case["in_off"], case["n"])
        inp.copy_(_plain_input(case, seed))
        state.update(inp=inp, out=_view(DTYPES[case["out_dt"]], case["out_off"], case["n"]))
    elif op in ("csr", "softmax"):
        offs = _offsets(case, seed)
        total = int(offs[-1])
        if op == "csr":
            inp = _lognormal(total, seed, 1.0).to(DTYPES[case["in_dt"]])
            out = torch.empty(total, dtype=DTYPES[case["out_dt"]], device="cuda")
        else:
            inp = torch.empty(total, device="cuda").normal_(0.0, 2.0, generator=_gen(seed))
            out = torch.empty_like(inp)
            state["lse"] = torch.empty(case["rows"], device="cuda")
        state["ctx"].batch_reserve(case["rows"], total)
        state.update(inp=inp, out=out, offsets=torch.from_numpy(offs).cuda())
    elif op == "rows":
        pairs = []
        for k, n in enumerate(_lengths(case)):
            x = _row_input(k, int(n), seed)
            pairs.append((torch.empty(int(n), dtype=DTYPES[MIX[k % len(MIX)][1]], device="cuda"), x))
        state["ctx"].batch_reserve(case["rows"], sum(x.numel() for _, x in pairs))
        state["pairs"] = pairs
    else:
        logp, target, weight = _nll_inputs(case, seed)
        want = case["n"] if case["reduction"] == "none" else 1
        state.update(logp=logp, target=target, weight=weight, out=torch.empty(want, device="cuda"),
                     total_weight=None if case["reduction"] == "none" else torch.empty(1, device="cuda"))
    return state


# ---- one pass ------------------------------------------------------------------------------


def run(state):
    case, ctx = state["case"], state["ctx"]
    op = case["op"]
    if op == "plain":
        return ctx.normalize(state["out"], state["inp"], accum=case["accum"])
    if op == "csr":
        return ctx.normalize_batched(state["out"], state["inp"], state["offsets"], accum=case["accum"])
    if op == "softmax":
        return [ctx.softmax_batched(state["out"], state["inp"], state["offsets"], lse=state["lse"]), state["lse"]]
    if op == "rows":
        ctx.normalize_rows(state["pairs"], accum=case["accum"])
        return [out for out, _ in state["pairs"]]
    out = api.nll_loss(state["logp"], state["target"], state["weight"], reduction=case["reduction"],
                       accum=case["accum"], out=state["out"], total_weight=state["total_weight"], ctx=ctx)
    return [out, state["total_weight"]]


# ---- what a pass cannot do without --------------------------------------------------------------


def work(case):
    op = case["op"]
    if op == "plain":
        n = case["n"]
        return {"bytes": n * (SIZE[case["in_dt"]] + SIZE[case["out_dt"]]), "flops": 2 * n}
    if op == "nll":
        # a target and one gathered log-probability per sample, the weights once, the outputs
        n, outs = case["n"], case["n"] if case["reduction"] == "none" else 2
        return {"bytes": 12 * n + (4 * case["c"] if case["weight"] else 0) + 4 * outs, "flops": 3 * n}
    rows, lengths = case["rows"], _lengths(case)
    total = int(lengths.sum())
    if op == "rows":
        moved = sum(int(n) * sum(SIZE[t] for t in MIX[k % len(MIX)]) for k, n in enumerate(lengths))
        return {"bytes": moved + 32 * rows, "flops": 2 * total}
    if op == "csr":
        return {"bytes": total * (SIZE[case["in_dt"]] + SIZE[case["out_dt"]]) + 8 * (rows + 1), "flops": 2 * total}
    return {"bytes": 8 * total + 12 * rows + 8, "flops": 6 * total}


# ---- the same in 64 bits ------------------------------------------------------------------------


def _per_row(x, offs, values):
    """Each element's row value from values[row]."""
    lengths = torch.from_numpy(np.diff(offs)).cuda()
    return torch.repeat_interleave(values, lengths, output_size=x.numel())


def _row_reduce(x, offs, kind):
    """Each row's sum or maximum (no row is empty)."""
    rows = offs.size - 1
    if rows <= 8192:  # few rows, long ones among them: one call each
        f = torch.sum if kind == "sum" else torch.amax
        return torch.stack([f(x[offs[r]:offs[r + 1]]) for r in range(rows)])
    ids = _per_row(x, offs, torch.arange(rows, device="cuda"))
    if kind == "sum":
        return torch.zeros(rows, dtype=x.dtype, device="cuda").index_add_(0, ids, x)
    return torch.full((rows,), -math.inf, dtype=x.dtype, device="cuda").scatter_reduce_(0, ids, x, "amax")


def exact(case, seed):
    op = case["op"]
    if op == "plain":
        x = _plain_input(case, seed).double()
        return x.div_(x.sum())
    if op == "csr":
        offs = _offsets(case, seed)
        x = _lognormal(int(offs[-1]), seed, 1.0).to(DTYPES[case["in_dt"]]).double()
        return x.div_(_per_row(x, offs, _row_reduce(x, offs, "sum")))
    if op == "softmax":
        offs = _offsets(case, seed)
        x = torch.empty(int(offs[-1]), device="cuda").normal_(0.0, 2.0, generator=_gen(seed)).double()
        top = _row_reduce(x, offs, "max")
        e = x.sub_(_per_row(x, offs, top)).exp_()
        sums = _row_reduce(e, offs, "sum")
        return [e.div_(_per_row(e, offs, sums)), top + sums.log()]
    if op == "rows":
        outs = []
        for k, n in enumerate(_lengths(case)):
            x = _row_input(k, int(n), seed).double()
            outs.append(x.div_(x.sum()))
        return outs
    logp, target, weight = _nll_inputs(case, seed)
    keep = target != -100
    t = target.clamp(min=0)
    w = (weight.double()[t] if weight is not None else torch.ones(case["n"], dtype=torch.float64, device="cuda")) * keep
    loss = -w * logp.gather(1, t[:, None])[:, 0].double()
    if case["reduction"] == "none":
        return [loss, None]
    total, wsum = loss.sum().reshape(1), w.sum().reshape(1)
    return [total / wsum if case["reduction"] == "mean" else total, wsum]
