"""Performance cases: the calls a user of this library makes, over the range of their sizes.

A case is a plain dict.  `listed()` names the standing ones, `draw(rng)` makes one more of the
same ranges, `prepare` makes what a program holds before the call (inputs, outputs, a plan),
`run` is one pass through the public entry points, `work` is what that pass cannot do without,
`tolerance` and `exact` say what its outputs must be.

Four operations:
  softmax    row softmax of packed score slices (uniform, ragged, one-row decode slices)
  backward   its gradient pass
  product    a batched bf16 matrix product ("nt" scores, "nn" context, "nt_softmax" scores with
             the row softmax in the same call)
  attention  one attention layer: nt_softmax product, then the context product
"""

import math
import random

import numpy as np
import torch

import paper_2002_07062_amd as bsm

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
SIGMA = 3.0  # scaled attention scores are drawn from N(0, 9), as in workloads.py


def _uniform(name, op, dtype, batch, rows, cols, call="plan", schedule="balanced", mask=0):
    """`batch` slices of rows x cols; mask > 0: slice s has its last 0..mask columns at -inf."""
    return {"name": name, "op": op, "dtype": dtype, "batch": batch, "rows": rows, "cols": cols,
            "mask": mask, "ragged": False, "call": call, "schedule": schedule}


def _ragged(name, op, dtype, batch, heads, rows, cols, step=1, square=False, call="plan",
            schedule="balanced", geometry=1):
    """`batch` slices, `heads` neighbours of one size; rows and cols drawn from [lo, hi] in
    steps of `step` (square: one length for both), packed one after the other."""
    return {"name": name, "op": op, "dtype": dtype, "batch": batch, "heads": heads,
            "rows_lo": rows[0], "rows_hi": rows[1], "cols_lo": cols[0], "cols_hi": cols[1],
            "step": step, "square": square, "geometry": geometry, "mask": 0, "ragged": True,
            "call": call, "schedule": schedule}


def _product(name, layout, dtype, batch, m, n, k, call="plan", schedule="balanced"):
    return {"name": name, "op": "product", "layout": layout, "dtype": dtype, "batch": batch,
            "m": m, "n": n, "k": k, "call": call, "schedule": schedule}


def _attention(name, batch, queries, keys, dim, temporal=False, schedule="balanced"):
    """bf16 Q (queries x dim), K and V (keys x dim) per batch index; temporal: plans that keep
    the probabilities in the Infinity Cache between the two calls."""
    return {"name": name, "op": "attention", "dtype": "bf16", "batch": batch, "m": queries,
            "n": keys, "k": dim, "temporal": temporal, "call": "plan", "schedule": schedule}


def listed():
    return [
        # the smallest call a program makes: a few short sequences, no plan kept by the caller
        _uniform("softmax_small_f32", "softmax", "f32", 8, 64, 64, call="oneshot"),
        # the headline workload: BERT's 384 score slices of 512 x 512
        _uniform("softmax_bert_f32", "softmax", "f32", 384, 512, 512),
        # the same in bf16 with key-padding masks baked in
        _uniform("softmax_masked_bf16", "softmax", "bf16", 384, 512, 512, mask=448),
        # slices of unrelated sizes, rows on 16-byte vectors (many models or layers in one batch)
        _ragged("softmax_ragged_f32", "softmax", "f32", 384, 1, (64, 1024), (64, 1024), step=8),
        # an unpadded batch: 32 sequences of any length x 12 heads, one-shot
        _ragged("softmax_varlen_bf16", "softmax", "bf16", 384, 12, (16, 512), (16, 512),
                square=True, call="oneshot"),
        # decode: one query row per sequence and head over a long cache, lengths all different
        _ragged("softmax_decode_bf16", "softmax", "bf16", 1024, 16, (1, 1), (1024, 32768)),
        # training: gradient of the headline workload
        _uniform("backward_bert_f32", "backward", "f32", 384, 512, 512),
        # training at long context
        _uniform("backward_long_f32", "backward", "f32", 32, 64, 16384),
        # BERT's score product
        _product("scores_bert_bf16", "nt", "bf16", 384, 512, 512, 64),
        # a context product over a sequence length that is no multiple of anything
        _product("context_odd_bf16", "nn", "bf16", 192, 333, 64, 333),
        # BERT's score product and softmax in one call
        _product("scores_softmax_bert_bf16", "nt_softmax", "bf16", 384, 512, 512, 64),
        # a long-context attention layer at head dimension 128
        _attention("attention_long_bf16", 32, 2048, 2048, 128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _length(rng, lo, hi):
    """A length over [lo, hi], half of the draws on a multiple of 8, the others anything."""
    n = _log_int(rng, lo, hi)
    if rng.random() < 0.5:
        n = (n + 4) // 8 * 8
    return max(lo, min(hi, n))


def draw(rng):
    case = _draw(rng)
    del case["name"]
    return case


def _draw(rng):
    kind = rng.choice(["uniform", "uniform", "ragged", "varlen", "decode", "product", "product",
                       "attention"])
    schedule = rng.choice(["balanced", "balanced", "balanced", "xcd"])
    call = rng.choice(["plan", "oneshot"])
    if kind in ("uniform", "ragged", "varlen", "decode"):
        op = rng.choice(["softmax", "softmax", "backward"])
        dtype = rng.choice(["f32", "bf16"])
        if kind == "uniform":
            cols = _length(rng, 16, 40000)
            elems = _log_int(rng, 1 << 15, 80_000_000)
            rows = _log_int(rng, 1, 1024)
            batch = max(1, min(20000, elems // (rows * cols)))
            if rows * cols * batch > 80_000_000:
                rows = max(1, 80_000_000 // (cols * batch))
            mask = cols // 2 if dtype == "bf16" and op == "softmax" and rng.random() < 0.5 else 0
            return _uniform("", op, dtype, batch, rows, cols, call, schedule, mask)
        geometry = rng.randrange(1, 1 << 30)
        if kind == "ragged":
            hi = _log_int(rng, 128, 1024)
            batch = _log_int(rng, 16, 300)
            step = rng.choice([1, 8])
            lo = 8 * rng.randint(1, 8)
            return _ragged("", op, dtype, batch, 1, (lo, hi), (lo, hi), step, False, call, schedule, geometry)
        if kind == "varlen":
            hi = _log_int(rng, 64, 512)
            heads = rng.choice([8, 12, 16])
            seqs = _log_int(rng, 2, 24)
            return _ragged("", op, dtype, heads * seqs, heads, (8, hi), (8, hi), 1, True, call, schedule,
                           geometry)
        heads = rng.choice([8, 16, 32])
        seqs = _log_int(rng, 4, 48)
        hi = _log_int(rng, 2048, 40000)
        return _ragged("", "softmax", dtype, heads * seqs, heads, (1, 1), (128, hi), 1, False, call,
                       schedule, geometry)
    dim = rng.choice([32, 64, 64, 80, 96, 128])
    m, n = _length(rng, 16, 2048), _length(rng, 16, 2048)
    batch = max(1, min(512, _log_int(rng, 1 << 16, 60_000_000) // (m * n)))
    if kind == "attention":
        return _attention("", batch, m, n, dim, rng.random() < 0.3, schedule)
    layout = rng.choice(["nt", "nn", "nt_softmax"])
    dtype = rng.choice(["f32", "bf16", "bf16"])
    if layout == "nn":
        return _product("", "nn", dtype, batch, m, dim, n, call, schedule)
    return _product("", layout, dtype, batch, m, n, dim, call, schedule)


# ---------------------------------------------------------------------------- geometry
def _sizes(case):
    """Rows and columns of every slice of a ragged case, and the offsets of their packing."""
    rng = random.Random(case["geometry"])

    def pick(lo, hi):
        return lo + case["step"] * rng.randint(0, (hi - lo) // case["step"])

    rows, cols, offsets, at = [], [], [], 0
    for s in range(case["batch"]):
        if s % case["heads"] == 0:
            c = pick(case["cols_lo"], case["cols_hi"])
            r = c if case["square"] else pick(case["rows_lo"], case["rows_hi"])
        rows.append(r)
        cols.append(c)
        offsets.append(at)
        at += r * c
    return rows, cols, offsets, at


def _elements(case):
    if case["ragged"]:
        return _sizes(case)[3]
    return case["batch"] * case["rows"] * case["cols"]


def _slices(case, *tensors):
    """The slices of flat tensors as 2-D (ragged) or one 3-D (uniform) view each."""
    if not case["ragged"]:
        shape = (case["batch"], case["rows"], case["cols"])
        yield tuple(t.view(shape) for t in tensors)
        return
    rows, cols, offsets, _ = _sizes(case)
    for r, c, o in zip(rows, cols, offsets):
        yield tuple(t[o:o + r * c].view(r, c) for t in tensors)


# ------------------------------------------------------------------------- state and runs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(n, dtype, g, sigma=1.0):
    x = torch.randn(n, device="cuda", generator=g)
    return (x if sigma == 1.0 else x.mul_(sigma)).to(DTYPES[dtype])


def _scores(case, g):
    x = _normal(_elements(case), case["dtype"], g, SIGMA)
    if case["mask"]:
        b, c = case["batch"], case["cols"]
        padded = torch.randint(0, case["mask"] + 1, (b, 1), device="cuda", generator=g)
        hide = torch.arange(c, device="cuda").expand(b, c) >= c - padded
        x.view(b, case["rows"], c).masked_fill_(hide[:, None, :], -math.inf)
    return x


def _geometry_args(case):
    if case["ragged"]:
        rows, cols, offsets, _ = _sizes(case)
        return {"rows": np.array(rows, np.int32), "cols": np.array(cols, np.int32),
                "slice_offsets": np.array(offsets, np.int64)}
    return {"rows": case["rows"], "cols": case["cols"], "batch": case["batch"]}


def prepare(case, seed):
    g = _generator(seed)
    state = {"case": case}
    b, dtype = case["batch"], case["dtype"]
    if case["op"] in ("softmax", "backward"):
        x = _scores(case, g)
        state["out"] = torch.empty_like(x)
        if case["op"] == "softmax":
            state["x"] = x
        else:  # the forward pass's output, and the gradient that arrives from above
            y = torch.empty_like(x)
            for xs, ys in _slices(case, x, y):
                ys.copy_(torch.softmax(xs.float(), dim=-1))
            state["y"] = y
            state["dy"] = _normal(x.numel(), dtype, g)
        state["geometry"] = _geometry_args(case)
        if case["call"] == "plan":
            state["plan"] = bsm.bsm_plan_create(dtype=dtype, schedule=case["schedule"],
                                                **state["geometry"])
        return state
    m, n, k = case["m"], case["n"], case["k"]
    if case["op"] == "attention":
        flags = {"flags": bsm.BSM_FLAG_TEMPORAL} if case["temporal"] else None
        state["alpha"] = 1.0 / math.sqrt(k)
        state["q"], state["k"], state["v"] = (_normal(b * r * k, "bf16", g) for r in (m, n, n))
        state["p"] = torch.empty(b * m * n, device="cuda", dtype=torch.bfloat16)
        state["o"] = torch.empty(b * m * k, device="cuda", dtype=torch.bfloat16)
        state["scores"] = bsm.bsm_gemm_plan_create(b, m, n, k, "nt_softmax", "bf16",
                                                   case["schedule"], topology=flags)
        state["context"] = bsm.bsm_gemm_plan_create(b, m, k, n, "nn", "bf16", case["schedule"],
                                                    topology=flags)
        return state
    state["alpha"] = 1.0 if case["layout"] == "nn" else 1.0 / math.sqrt(k)
    if case["layout"] == "nn":  # context: A holds softmax rows
        p = torch.softmax(torch.randn(b * m, k, device="cuda", generator=g).mul_(SIGMA), dim=-1)
        state["a"] = p.to(torch.bfloat16).view(-1)
    else:
        state["a"] = _normal(b * m * k, "bf16", g)
    state["b"] = _normal(b * n * k, "bf16", g)
    state["c"] = torch.empty(b * m * n, device="cuda", dtype=DTYPES[dtype])
    if case["call"] == "plan":
        state["plan"] = bsm.bsm_gemm_plan_create(b, m, n, k, case["layout"], dtype,
                                                 case["schedule"])
    return state


def run(state):
    case = state["case"]
    op, sched = case["op"], case["schedule"]
    if op == "softmax":
        if case["call"] == "plan":
            return bsm.bsm_plan_execute(state["plan"], state["x"], state["out"])
        return bsm.bsm_softmax(state["x"], state["out"], schedule=sched, **state["geometry"])
    if op == "backward":
        if case["call"] == "plan":
            return bsm.bsm_plan_execute_backward(state["plan"], state["y"], state["dy"], state["out"])
        return bsm.bsm_softmax_backward(state["y"], state["dy"], state["out"], schedule=sched,
                                        **state["geometry"])
    if op == "attention":
        bsm.bsm_gemm_execute(state["scores"], state["q"], state["k"], state["p"], state["alpha"])
        bsm.bsm_gemm_execute(state["context"], state["p"], state["v"], state["o"])
        return state["p"], state["o"]
    if case["call"] == "plan":
        return bsm.bsm_gemm_execute(state["plan"], state["a"], state["b"], state["c"], state["alpha"])
    return bsm.bsm_gemm(state["a"], state["b"], state["c"], case["batch"], case["m"], case["n"],
                        case["k"], case["layout"], state["alpha"], sched)


def work(case):
    es = 4 if case["dtype"] == "f32" else 2
    if case["op"] in ("softmax", "backward"):
        n = _elements(case)
        # forward: maximum, difference, exponential, sum, scale; backward: two products, two sums
        streams, per_element = (2, 5) if case["op"] == "softmax" else (3, 4)
        return {"bytes": streams * n * es, "flops": per_element * n}
    b, m, n, k = case["batch"], case["m"], case["n"], case["k"]
    if case["op"] == "attention":
        return {"bytes": b * 2 * (2 * m * k + 2 * n * k + m * n), "flops": b * (4 * m * n * k + 5 * m * n)}
    flops = 2 * b * m * n * k + (5 * b * m * n if case["layout"] == "nt_softmax" else 0)
    return {"bytes": b * (2 * (m * k + n * k) + es * m * n), "flops": flops}


# ----------------------------------------------------------------------------- correctness
def tolerance(case):
    # measured against exact() over the listed cases and drawn ones: bf16 outputs 1.5e-3 to
    # 1.7e-3 (one rounding to bf16 of every value; the attention layer's second output is of
    # the probabilities as its first call rounded them), fp32 outputs 0.7e-7 to 1.0e-7 (sums
    # of up to 32768 terms in some order, more in another order)
    return {"rel": 7e-3} if case["dtype"] == "bf16" else {"rel": 1e-6}


def exact(case, seed):
    state = prepare(case, seed)
    if case["op"] == "softmax":
        out = torch.empty(state["x"].numel(), device="cuda", dtype=torch.float64)
        for xs, os in _slices(case, state["x"], out):
            os.copy_(torch.softmax(xs.double(), dim=-1))
        return out
    if case["op"] == "backward":
        out = torch.empty(state["y"].numel(), device="cuda", dtype=torch.float64)
        for ys, gs, os in _slices(case, state["y"], state["dy"], out):
            y, dy = ys.double(), gs.double()
            os.copy_(y * (dy - (y * dy).sum(dim=-1, keepdim=True)))
        return out
    b, m, n, k = case["batch"], case["m"], case["n"], case["k"]

    def nt(x, y, alpha):
        x = x.view(b, m, k).double()
        return torch.bmm(x, y.view(b, n, k).double().transpose(1, 2).contiguous()).mul_(alpha)

    if case["op"] == "attention":
        p = torch.softmax(nt(state["q"], state["k"], state["alpha"]), dim=-1)
        # the context product is of the bf16 probabilities that the first call stored
        o = torch.bmm(p.to(torch.bfloat16).double(), state["v"].view(b, n, k).double())
        return p.view(-1), o.reshape(-1)
    if case["layout"] == "nn":
        c = torch.bmm(state["a"].view(b, m, k).double(), state["b"].view(b, k, n).double())
        return c.mul_(state["alpha"]).view(-1)
    c = nt(state["a"], state["b"], state["alpha"])
    return (torch.softmax(c, dim=-1) if case["layout"] == "nt_softmax" else c).view(-1)
