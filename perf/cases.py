"""Performance cases: the work a program has this library do, through its
public Python entry points, over the sizes, types and options in use.

Families (`kind`):
  ew      elementwise statements (float32, bfloat16 -> FP8, complex64, shifted
          reads); n from a launch-bound 256 to 2^28
  red     map-reduce to one value (dot, count, sum, max, complex dot)
  prec    compensated sums and scaled L2 norms of narrow storage formats
  scan    prefix scans (float32 and int32 -> int64, inclusive and exclusive)
  seg     segmented map-reduce over many uneven segments
  cg      conjugate-gradient iterations on the five-point model problem
  serve   a queue of map-reduce jobs drained by the default server
"""

import math

import numpy as np
import torch

import paper_1304_5553_amd as hm
from paper_1304_5553_amd import cg as hcg

# ---------------------------------------------------------------- statements
# op: (signature, statement)
EW = {
    "lincomb": ("float *z, const float *x, const float *y", "z[i] = 2.5f*x[i] - 0.5f*y[i]"),
    "hypot": ("float *z, const float *x, const float *y", "z[i] = sqrtf(x[i]*x[i] + y[i]*y[i])"),
    "diff": ("float *z, const float *x, const float *y", "z[i] = x[i] - y[i]"),
    "quantize": ("fp8_e4m3 *z, const bfloat16 *x, float s", "z[i] = s*x[i]"),
    "dequantize": ("bfloat16 *z, const fp8_e4m3 *x, float s", "z[i] = s*x[i]"),
    "stencil": ("float *z, const float *x",
                "z[i] = x[i] - 0.5f*((i >= 1 ? x[i-1] : 0.0f) + (i + 1 < n ? x[i+1] : 0.0f))"),
    "caxpby": ("complex64 *z, complex64 a, const complex64 *x, complex64 b, const complex64 *y",
               "z[i] = a*x[i] + b*y[i]"),
}
EW_BYTES = {"lincomb": 12, "hypot": 12, "diff": 8, "quantize": 3, "dequantize": 3, "stencil": 8, "caxpby": 24}
EW_FLOPS = {"lincomb": 3, "hypot": 4, "diff": 1, "quantize": 1, "dequantize": 1, "stencil": 4, "caxpby": 14}
CA, CB = 0.75 - 1.25j, -0.5 + 0.25j

# op: (signature, map expression, combine, neutral element)
RED = {
    "dot": ("float: const float *x, const float *y", "x[i]*y[i]", "a+b", "0"),
    "sumf": ("float: const float *x", "x[i]", "a+b", "0"),
    "max": ("float: const float *x", "x[i]", "max(a,b)", "-INFINITY"),
    "count": ("long: const int *k", "k[i] % 7 == 3", "a+b", "0"),
    "sum": ("long: const int *k", "k[i]", "a+b", "0"),
    "cdot": ("complex64: const complex64 *x, const complex64 *y", "conj(x[i]) * y[i]", "a+b", "0"),
}
RED_BYTES = {"dot": 8, "sumf": 4, "max": 4, "count": 4, "sum": 4, "cdot": 16}
RED_FLOPS = {"dot": 2, "sumf": 1, "max": 1, "count": 3, "sum": 1, "cdot": 8}

STORAGE = {"float": torch.float32, "bfloat16": torch.bfloat16, "half": torch.float16,
           "fp8_e4m3": torch.float8_e4m3fn}


def listed():
    return [
        # one small fused statement, as in the inner loop of a script: the call's latency
        {"name": "lincomb_4k", "kind": "ew", "op": "lincomb", "n": 4096, "view": 0},
        # the streaming statement of the headline workload at its full size
        {"name": "lincomb_2e28", "kind": "ew", "op": "lincomb", "n": 1 << 28, "view": 0},
        # forward difference of one signal given as the two views x[1:] and x[:-1]
        {"name": "diff_views", "kind": "ew", "op": "diff", "n": 50_000_003, "view": 1},
        # quantising an activation tensor of odd size for storage
        {"name": "quantize_fp8", "kind": "ew", "op": "quantize", "n": (1 << 26) + 5, "view": 0},
        # the small dot product (one map-reduce over 2^20 pairs): two short kernels
        {"name": "dot_1m", "kind": "red", "op": "dot", "n": 1 << 20, "view": 0},
        # the counting map-reduce of the headline workload at its full size
        {"name": "count_2e28", "kind": "red", "op": "count", "n": 1 << 28, "view": 0},
        # L2 norm of a large bfloat16 tensor (gradient clipping)
        {"name": "norm_bf16_2e27", "kind": "prec", "op": "norm", "fmt": "bfloat16", "n": 1 << 27},
        # cumulative sum of a long float signal
        {"name": "scan_f32_2e28", "kind": "scan", "op": "sumf", "n": 1 << 28, "exclusive": False},
        # exclusive offsets from a list of counts (int32 -> int64), an ordinary odd size
        {"name": "scan_i64_100k", "kind": "scan", "op": "sum", "n": 100_003, "exclusive": True},
        # 4096 uneven segments in one call (ragged batch), mean 2^14 elements
        {"name": "segments_4096", "kind": "seg", "op": "sumf", "nseg": 4096, "median": 4096},
        # twenty solver iterations on a mid-size grid, issued one call after another
        {"name": "cg_1024x768", "kind": "cg", "nx": 1024, "ny": 768, "iters": 20},
        # a queue of 64 mixed jobs handed to the server at once
        {"name": "serve_64", "kind": "serve", "jobs": 64, "log2_max": 20},
    ]


def _log_uniform(rng, lo, hi):
    n = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    return n if rng.random() < 0.25 else n | 1


def draw(rng):
    kind = rng.choice(["ew", "ew", "ew", "red", "red", "prec", "scan", "scan", "seg", "cg", "serve"])
    if kind == "ew":
        op = rng.choice(sorted(EW))
        n = _log_uniform(rng, 256, (1 << 28) * 12 // EW_BYTES[op] // (4 if EW_BYTES[op] <= 3 else 1))
        return {"kind": kind, "op": op, "n": n, "view": 1 if op == "diff" else rng.choice([0, 0, 0, 1])}
    if kind == "red":
        op = rng.choice(sorted(RED))
        return {"kind": kind, "op": op, "n": _log_uniform(rng, 256, (1 << 28) * 4 // RED_BYTES[op]),
                "view": rng.choice([0, 0, 0, 1])}
    if kind == "prec":
        return {"kind": kind, "op": rng.choice(["norm", "sum"]), "fmt": rng.choice(sorted(STORAGE)),
                "n": _log_uniform(rng, 1 << 20, 1 << 27)}
    if kind == "scan":
        op = rng.choice(["sumf", "sum"])
        return {"kind": kind, "op": op, "n": _log_uniform(rng, 256, 1 << (28 if op == "sumf" else 27)),
                "exclusive": rng.random() < 0.5}
    if kind == "seg":
        nseg = _log_uniform(rng, 16, 16384)
        return {"kind": kind, "op": rng.choice(["sumf", "max", "dot"]), "nseg": nseg,
                "median": _log_uniform(rng, 32, min(16384, max(64, (1 << 24) // nseg)))}
    if kind == "cg":
        return {"kind": kind, "nx": _log_uniform(rng, 48, 2048), "ny": _log_uniform(rng, 48, 2048),
                "iters": rng.choice([4, 10, 20])}
    return {"kind": kind, "jobs": _log_uniform(rng, 8, 256), "log2_max": rng.choice([16, 18, 20])}


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(g, n, lo, hi, dtype=torch.float32):
    return torch.empty(n, dtype=dtype, device="cuda").uniform_(lo, hi, generator=g)


def _normal(g, n):
    return torch.empty(n, dtype=torch.float32, device="cuda").normal_(0.0, 1.0, generator=g)


def _narrow(fmt, v):
    return v.clamp(-448.0, 448.0).to(STORAGE[fmt]) if fmt == "fp8_e4m3" else v.to(STORAGE[fmt])


def _complex(g, n):
    return torch.view_as_complex(_uniform(g, 2 * n, -0.5, 1.0).view(n, 2))


def _ew_inputs(case, seed):
    """The statement's input arrays, by argument name."""
    g, n, op, view = _gen(seed), case["n"], case["op"], case["view"]
    if op == "diff":                       # two views of one signal
        s = _uniform(g, n + 1, -1.0, 1.0)
        return {"x": s[1:], "y": s[:-1]}
    if op in ("lincomb", "hypot"):
        return {"x": _uniform(g, n + view, -1.0, 1.0)[view:], "y": _uniform(g, n, -1.0, 1.0)}
    if op == "stencil":
        return {"x": _uniform(g, n + view, -1.0, 1.0)[view:]}
    if op == "caxpby":
        return {"x": _complex(g, n + view)[view:], "y": _complex(g, n)}
    x = _normal(g, n + view)
    if op == "quantize":
        return {"x": _narrow("bfloat16", x)[view:]}
    return {"x": _narrow("fp8_e4m3", x.mul_(56.0))[view:]}


QUANT_SCALE, DEQUANT_SCALE = 56.0, 1.0 / 56.0


def _red_inputs(case, seed):
    g, n, op, view = _gen(seed), case["n"], case["op"], case["view"]
    if op in ("count", "sum"):
        return {"k": torch.randint(0, 1 << 20, (n + view,), dtype=torch.int32, device="cuda", generator=g)[view:]}
    if op == "cdot":
        return {"x": _complex(g, n + view)[view:], "y": _complex(g, n)}
    if op == "max":
        return {"x": _normal(g, n + view)[view:]}
    x = {"x": _uniform(g, n + view, -0.5, 1.0)[view:]}
    if op == "dot":
        x["y"] = _uniform(g, n, -0.5, 1.0)
    return x


def _prec_input(case, seed):
    g, n = _gen(seed), case["n"]
    if case["op"] == "norm":               # gradients: centred, one scale per tensor
        v = _normal(g, n)
    else:                                  # probabilities / losses: non-negative
        v = _uniform(g, n, 0.0, 1.0)
    return _narrow(case["fmt"], v)


def _segments(case, seed):
    """Offsets (host int64) of `nseg` lognormal segments clipped to [1, 2^20]."""
    rng = np.random.default_rng(int(seed))
    sigma = math.sqrt(2.0 * math.log(4.0))
    lens = np.clip(np.rint(rng.lognormal(math.log(case["median"]), sigma, case["nseg"])), 1, 1 << 20)
    off = np.zeros(case["nseg"] + 1, np.int64)
    np.cumsum(lens.astype(np.int64), out=off[1:])
    return off


def _seg_inputs(case, seed):
    off = _segments(case, seed)
    g, total = _gen(seed), int(off[-1])
    x = {"x": _normal(g, total) if case["op"] == "max" else _uniform(g, total, -0.5, 1.0)}
    if case["op"] == "dot":
        x["y"] = _uniform(g, total, -0.5, 1.0)
    return torch.from_numpy(off).cuda(), x


def _cg_input(case, seed):
    return _uniform(_gen(seed), case["nx"] * case["ny"], -1.0, 1.0)


POOL = 1 << 21


def _serve_inputs(case, seed):
    """The resident pool (x, y ~ U[-1, 1], w ~ U[0, 1), float32 and bfloat16)
    and the jobs as host records (n, template, bfloat16 flag, offset)."""
    g = _gen(seed)
    pool = {"x": _uniform(g, POOL, -1.0, 1.0), "y": _uniform(g, POOL, -1.0, 1.0), "w": _uniform(g, POOL, 0.0, 1.0)}
    low = {k: v.to(torch.bfloat16) for k, v in pool.items()}
    rng = np.random.default_rng(int(seed))
    m = case["jobs"]
    n = np.floor(2.0 ** rng.uniform(10, case["log2_max"], m)).astype(np.int64)
    return pool, low, {"n": n, "tmpl": rng.integers(0, 8, m), "bf16": rng.random(m) < 0.5,
                       "offset": (rng.random(m) * (POOL - n + 1)).astype(np.int64)}


# ---------------------------------------------------------------- prepare / run
def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "n": case.get("n")}
    if kind == "ew":
        sig, stmt = EW[case["op"]]
        a = _ew_inputs(case, seed)
        s["k"] = hm.compile(stmt, sig)
        zt = {"quantize": torch.float8_e4m3fn, "dequantize": torch.bfloat16,
              "caxpby": torch.complex64}.get(case["op"], torch.float32)
        z = torch.empty(case["n"], dtype=zt, device="cuda")
        s["out"] = z
        if case["op"] == "quantize":
            s["args"] = [z, a["x"], QUANT_SCALE]
        elif case["op"] == "dequantize":
            s["args"] = [z, a["x"], DEQUANT_SCALE]
        elif case["op"] == "caxpby":
            s["args"] = [z, CA, a["x"], CB, a["y"]]
        else:
            s["args"] = [z, *a.values()]
    elif kind == "red":
        sig, expr, s["combine"], s["neutral"] = RED[case["op"]]
        s["k"] = hm.compile(expr, sig)
        hm.prepare_reduce(s["k"], s["combine"], s["neutral"])
        s["args"] = list(_red_inputs(case, seed).values())
        s["out"] = torch.empty((), dtype=hm.torch_dtype(s["k"].result_dtype), device="cuda")
    elif kind == "prec":
        s["k"] = hm.compile("x[i]", f"float: const {case['fmt']} *x")
        s["args"] = [_prec_input(case, seed)]
        s["out"] = torch.empty((), dtype=torch.float64, device="cuda")
    elif kind == "scan":
        sig, expr, s["combine"], s["neutral"] = RED[case["op"]]
        s["k"] = hm.compile(expr, sig)
        s["args"] = list(_red_inputs(dict(case, view=0), seed).values())
        s["out"] = torch.empty(case["n"], dtype=hm.torch_dtype(s["k"].result_dtype), device="cuda")
    elif kind == "seg":
        sig, expr, s["combine"], s["neutral"] = RED[case["op"]]
        s["k"] = hm.compile(expr, sig)
        s["offsets"], a = _seg_inputs(case, seed)
        s["args"], s["total"] = list(a.values()), a["x"].numel()
        s["out"] = torch.empty(case["nseg"], dtype=torch.float32, device="cuda")
    elif kind == "cg":
        s["b"] = _cg_input(case, seed)
        s["solver"] = hcg.PoissonCG(case["nx"], case["ny"])
    else:
        pool, low, recs = _serve_inputs(case, seed)
        s["server"] = hm.Server()
        s["keep"] = (pool, low)
        s["out"] = torch.empty(case["jobs"], dtype=torch.float64, device="cuda")
        jobs = s["server"].jobs(case["jobs"])
        for j in range(case["jobs"]):
            src, size = (low, 2) if recs["bf16"][j] else (pool, 4)
            at = int(recs["offset"][j]) * size
            for name in ("x", "y", "w"):
                jobs[name][j] = src[name].data_ptr() + at
            jobs["dtype"][j] = hm.hipmr.BF16 if recs["bf16"][j] else hm.hipmr.F32
            jobs["out"][j] = s["out"].data_ptr() + 8 * j
        jobs["n"], jobs["tmpl"], jobs["a"], jobs["b"] = recs["n"], recs["tmpl"], 2.5, -0.5
        s["jobs"] = jobs
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "ew":
        hm.elementwise(s["k"], s["n"], s["args"])
        return s["out"]
    if kind == "red":
        return hm.reduce(s["k"], None, s["combine"], s["neutral"], s["n"], s["args"], s["out"])
    if kind == "prec":
        f = hm.norm2 if case["op"] == "norm" else hm.reduce_compensated
        return f(s["k"], s["n"], s["args"], out=s["out"])
    if kind == "scan":
        return hm.scan(s["k"], s["combine"], s["neutral"], s["n"], s["args"], s["out"], exclusive=case["exclusive"])
    if kind == "seg":
        return hm.reduce_segmented(s["k"], s["combine"], s["neutral"], s["offsets"], s["total"], s["args"], s["out"])
    if kind == "cg":
        x = s["solver"].solve(s["b"], case["iters"])
        return {"x": x, "r": s["solver"].r, "p": s["solver"].p, "rr": s["solver"].rr}
    done = s["server"].run_schedule(s["jobs"])
    return {"out": s["out"], "status": done["status"]}


# ---------------------------------------------------------------- work
def work(case):
    kind = case["kind"]
    n = case.get("n", 0)
    if kind == "ew":
        return {"bytes": EW_BYTES[case["op"]] * n, "flops": EW_FLOPS[case["op"]] * n}
    if kind == "red":
        return {"bytes": RED_BYTES[case["op"]] * n, "flops": RED_FLOPS[case["op"]] * n}
    if kind == "prec":
        size = {"float": 4, "bfloat16": 2, "half": 2, "fp8_e4m3": 1}[case["fmt"]]
        return {"bytes": size * n, "flops": 2 * n}
    if kind == "scan":
        return {"bytes": (8 if case["op"] == "sumf" else 12) * n, "flops": n}
    if kind == "seg":
        total = int(_segments(case, 1)[-1])
        return {"bytes": RED_BYTES[case["op"]] * total + 12 * case["nseg"], "flops": RED_FLOPS[case["op"]] * total}
    if kind == "cg":                       # x, r and p read and written once per iteration
        m = case["nx"] * case["ny"] * case["iters"]
        return {"bytes": 24 * m, "flops": 18 * m}
    m = case["jobs"] * (2 ** case["log2_max"] - 2 ** 10) / (math.log(2) * (case["log2_max"] - 10))   # mean size
    return {"bytes": 4.1 * m, "flops": 1.9 * m}


# ---------------------------------------------------------------- exact values
def _wide(t):
    return t.to(torch.complex128 if t.is_complex() else torch.float64)


def _exact_ew(case, seed):
    a = {k: _wide(v) for k, v in _ew_inputs(case, seed).items()}
    op, x = case["op"], a["x"]
    if op == "lincomb":
        return 2.5 * x - 0.5 * a["y"]
    if op == "hypot":
        return torch.sqrt(x * x + a["y"] * a["y"])
    if op == "diff":
        return x - a["y"]
    if op == "quantize":
        return (QUANT_SCALE * x).clamp(-448.0, 448.0)
    if op == "dequantize":
        return float(np.float32(DEQUANT_SCALE)) * x
    if op == "caxpby":
        return CA * x + CB * a["y"]
    z = x.clone()
    z[1:] -= 0.5 * x[:-1]
    z[:-1] -= 0.5 * x[1:]
    return z


def _exact_map(op, a):
    if op == "dot":
        return _wide(a["x"]) * _wide(a["y"])
    if op == "cdot":
        return _wide(a["x"]).conj() * _wide(a["y"])
    return _wide(a["x"])


def _exact_cg(case, seed):
    b = _wide(_cg_input(case, seed))
    ny, nx = case["ny"], case["nx"]

    def apply(v):
        g = v.view(ny, nx)
        q = 4.0 * g
        q[:, 1:] -= g[:, :-1]
        q[:, :-1] -= g[:, 1:]
        q[1:] -= g[:-1]
        q[:-1] -= g[1:]
        return q.reshape(-1)
    x, r, p = torch.zeros_like(b), b.clone(), b.clone()
    rr = r.dot(r)
    for _ in range(case["iters"]):
        q = apply(p)
        alpha = rr / p.dot(q)
        x += alpha * p
        r -= alpha * q
        nxt = r.dot(r)
        p = r + (nxt / rr) * p
        rr = nxt
    return {"x": x, "r": r, "p": p, "rr": rr.reshape(1)}


def _exact_serve(case, seed):
    pool, low, recs = _serve_inputs(case, seed)
    out = []
    for j in range(case["jobs"]):
        src = low if recs["bf16"][j] else pool
        o, n = int(recs["offset"][j]), int(recs["n"][j])
        x, y, w = (_wide(src[k][o:o + n]) for k in ("x", "y", "w"))
        out.append([lambda: x.sum(), lambda: x.dot(y), lambda: x.dot(x).sqrt(), lambda: x.max(),
                    lambda: (2.5 * x - 0.5 * y).sum(), lambda: (x > 0).sum(), lambda: x.dot(x),
                    lambda: w.dot(x) / w.sum()][int(recs["tmpl"][j])]().double().item())
    return {"out": torch.tensor(out, dtype=torch.float64), "status": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "ew":
        return _exact_ew(case, seed)
    if kind == "red":
        a = _red_inputs(case, seed)
        if case["op"] in ("count", "sum"):
            return None                    # whole numbers
        v = _exact_map(case["op"], a)
        return v.max() if case["op"] == "max" else v.sum()
    if kind == "prec":
        v = _prec_input(case, seed).to(torch.float32).double()
        return torch.sqrt((v * v).sum()) if case["op"] == "norm" else v.sum()
    if kind == "scan":
        if case["op"] == "sum":
            return None                    # whole numbers
        v = torch.cumsum(_wide(_red_inputs(dict(case, view=0), seed)["x"]), 0)
        if case["exclusive"]:
            v = torch.cat([v.new_zeros(1), v[:-1]])
        return v
    if kind == "seg":
        off, a = _seg_inputs(case, seed)
        v = _exact_map(case["op"], a)
        ids = torch.repeat_interleave(torch.arange(case["nseg"], device="cuda"), off[1:] - off[:-1])
        if case["op"] == "max":
            return torch.full((case["nseg"],), -math.inf, dtype=torch.float64,
                              device="cuda").scatter_reduce_(0, ids, v, "amax")
        return torch.zeros(case["nseg"], dtype=torch.float64, device="cuda").index_add_(0, ids, v)
    if kind == "cg":
        return _exact_cg(case, seed)
    return _exact_serve(case, seed)
