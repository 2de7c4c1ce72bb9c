"""Performance cases of the GEMM library: what a program calls it with.

Every case goes through the Python binding's public entry points (``gemm``,
``gemm_ex``, ``gemm_split``, ``Plan.launch``, ``gemm_batched``, ``daxpy``).
A case is a dict of plain values; ``prepare`` builds what a caller has in hand
before the call, ``run`` makes one call and returns its whole output, ``work``
gives the bytes and operations one call cannot do without, and ``exact`` the
same result from plain torch in 64 bits.
"""

from __future__ import annotations

import math
import random

import torch

import paper_1602_08477_amd as mg

_SCALARS = ((1.0, 1.0), (1.5, 0.5), (1.0, 0.0))


def _gemm(name, m, n, k, dtype="f64", ta=False, tb=False, pad=1, alpha=1.0, beta=1.0):
    """One dense product; ``pad``: row pitches are rounded up to a multiple of
    it (1: tightly packed rows, whatever their length)."""
    return {"name": name, "kind": "gemm", "m": m, "n": n, "k": k, "dtype": dtype, "ta": ta,
            "tb": tb, "pad": pad, "alpha": alpha, "beta": beta}


def _split(name, m, n, k, algo, alpha=1.0, beta=1.0):
    return {"name": name, "kind": "split", "m": m, "n": n, "k": k, "algo": algo, "alpha": alpha,
            "beta": beta}


def _batch(name, count, lo, hi, dtype="f64", algo="native", call="plan"):
    return {"name": name, "kind": "batch", "count": count, "lo": lo, "hi": hi, "dtype": dtype,
            "algo": algo, "call": call}


def listed():
    return [
        # the smallest single products of the request mix (n in [32, 2048]): latency
        _gemm("gemm_f64_64", 64, 64, 64),
        # the single-product workload of the tests and the bench
        _gemm("gemm_f64_512", 512, 512, 512, alpha=1.5, beta=0.5),
        # an ordinary square product; the size sweep's middle
        _gemm("gemm_f64_2048", 2048, 2048, 2048),
        # the headline product of the bench
        _gemm("gemm_f64_8192", 8192, 8192, 8192),
        # tightly packed matrices with odd extents: rows only 8-byte aligned
        _gemm("gemm_f64_odd", 1531, 1033, 2047),
        # single precision, ordinary size
        _gemm("gemm_f32_2048", 2048, 2048, 2048, dtype="f32"),
        # A^T B over a long common extent (normal equations, weight gradients):
        # a small output and a long sum
        _gemm("gemm_tn_long_k", 384, 384, 8192, ta=True, beta=0.0),
        # FP64 rebuilt from INT8 slices at the size the bench compares it at
        _split("split_i8_4096", 4096, 4096, 4096, "i8"),
        # uneven batch in one launch: the 2000-problem workload, both types
        _batch("batched_f64_2000", 2000, 16, 512),
        _batch("batched_f32_2000", 2000, 16, 512, dtype="f32"),
        # the same batch through the split-precision path, one-shot call
        _batch("batched_i8_2000", 2000, 16, 512, algo="i8", call="oneshot"),
        # the vector kernel at the bench's length
        {"name": "daxpy_2p27", "kind": "daxpy", "n": 1 << 27, "shift": 0, "alpha": 1.25},
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    u = rng.random()
    alpha, beta = rng.choice(_SCALARS)
    if u < 0.55:  # single products: any shape from 32 to 8192 per extent, k to 16384
        while True:
            m, n = _log_int(rng, 32, 8192), _log_int(rng, 32, 8192)
            k = _log_int(rng, 32, 16384)
            if m * n * k <= 1 << 36:
                break
        if rng.random() < 0.4:  # sizes a program picks itself are often round
            m, n, k = (max(32, x // 32 * 32) for x in (m, n, k))
        ta, tb = rng.random() < 0.25, rng.random() < 0.25
        c = _gemm("", m, n, k, rng.choice(("f64", "f64", "f32")), ta, tb,
                  rng.choice((1, 1, 16)), alpha, beta)
    elif u < 0.7:  # split precision: 64 to 4096 per extent
        m, n, k = (_log_int(rng, 64, 4096) for _ in range(3))
        c = _split("", m, n, k, rng.choice(("i8", "i8", "bf16")), alpha, beta)
    elif u < 0.92:  # batches: 16 to 2000 problems, extents up to 512
        algo = rng.choice(("native", "native", "i8", "bf16"))
        dtype = rng.choice(("f64", "f32")) if algo == "native" else "f64"
        call = rng.choice(("plan", "oneshot")) if algo == "native" else "oneshot"
        c = _batch("", _log_int(rng, 16, 2000), rng.choice((16, 32, 64)),
                   rng.choice((128, 256, 512)), dtype, algo, call)
    else:
        c = {"name": "", "kind": "daxpy", "n": _log_int(rng, 1000, 1 << 27),
             "shift": rng.choice((0, 0, 1)), "alpha": 1.25}
    del c["name"]
    return c


# ------------------------------------------------------------------- inputs
_DTYPES = {"f64": torch.float64, "f32": torch.float32}
_ALGOS = {"native": mg.NATIVE, "i8": mg.SPLIT_I8, "bf16": mg.SPLIT_BF16}


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _mat(rows, cols, dtype, g, pad=1):
    """Uniform [-1, 1) values, rows of pitch ``cols`` rounded up to ``pad``."""
    ld = -(-cols // pad) * pad
    t = torch.empty(rows, ld, dtype=dtype, device="cuda")
    t.uniform_(-1.0, 1.0, generator=g)
    return t[:, :cols]


def _spread(rows, cols, g):
    """(2u - 1) * 2^e, e uniform in [-20, 20]: values of widely spread exponents."""
    t = torch.empty(rows, cols, dtype=torch.float64, device="cuda").uniform_(-1.0, 1.0, generator=g)
    e = torch.randint(-20, 21, (rows, cols), device="cuda", generator=g)
    return torch.ldexp(t, e)


def _operands(case, seed):
    g = _gen(seed)
    m, n, k = case["m"], case["n"], case["k"]
    if case["kind"] == "split":
        return _spread(m, k, g), _spread(k, n, g), _spread(m, n, g)
    dt, pad = _DTYPES[case["dtype"]], case["pad"]
    A = _mat(k, m, dt, g, pad) if case["ta"] else _mat(m, k, dt, g, pad)
    B = _mat(n, k, dt, g, pad) if case["tb"] else _mat(k, n, dt, g, pad)
    return A, B, _mat(m, n, dt, g, pad)


def _batch_shapes(case):
    """Log-uniform extents: the shapes belong to the case, the values to the seed."""
    r = random.Random(case["count"])
    return [tuple(_log_int(r, case["lo"], case["hi"]) for _ in range(3))
            for _ in range(case["count"])]


def _batch_operands(case, seed):
    """Views of three flat buffers (all A, all B, all C), tightly packed."""
    g = _gen(seed)
    dt = _DTYPES[case["dtype"]]
    shapes = _batch_shapes(case)
    flat = []
    for rows, cols in ((0, 2), (2, 1), (0, 1)):
        total = sum(-(-s[rows] * s[cols] // 16) * 16 for s in shapes)
        flat.append(torch.empty(total, dtype=dt, device="cuda").uniform_(-1.0, 1.0, generator=g))
    views, at = [], [0, 0, 0]
    for m, n, k in shapes:
        v = []
        for i, (r, c) in enumerate(((m, k), (k, n), (m, n))):
            v.append(flat[i][at[i]:at[i] + r * c].view(r, c))
            at[i] += -(-r * c // 16) * 16
        views.append(v)
    return flat, views


def _axpy_operands(case, seed):
    g = _gen(seed)
    n, shift = case["n"], case["shift"]
    x = torch.empty(n + shift, dtype=torch.float64, device="cuda").uniform_(-1, 1, generator=g)
    y = torch.empty(n + shift, dtype=torch.float64, device="cuda").uniform_(-1, 1, generator=g)
    return x[shift:], y[shift:]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "daxpy":
        x, y = _axpy_operands(case, seed)
        return {"kind": kind, "alpha": case["alpha"], "x": x, "y": y}
    if kind == "batch":
        flat, views = _batch_operands(case, seed)
        probs = mg.problems_array([mg.problem(A, B, C, 1.0, 1.0) for A, B, C in views])
        dt = mg.F64 if case["dtype"] == "f64" else mg.F32
        s = {"kind": kind, "call": case["call"], "dtype": dt, "algo": _ALGOS[case["algo"]],
             "probs": probs, "flat": flat}
        if case["call"] == "plan":
            s["plan"] = mg.Plan(dt, probs, keep=flat)
        return s
    A, B, C = _operands(case, seed)
    s = {"kind": kind, "A": A, "B": B, "C": C, "alpha": case["alpha"], "beta": case["beta"]}
    if kind == "split":
        algo = _ALGOS[case["algo"]]
        s["algo"] = algo
        s["ws"] = mg.split_workspace(algo, mg.split_default_slices(algo), case["m"], case["n"],
                                     case["k"])
    else:
        s["ta"], s["tb"] = case["ta"], case["tb"]
    return s


def run(s):
    kind = s["kind"]
    if kind == "gemm":
        if s["ta"] or s["tb"]:
            return mg.gemm_ex(s["A"], s["B"], s["C"], s["alpha"], s["beta"], s["ta"], s["tb"])
        return mg.gemm(s["A"], s["B"], s["C"], s["alpha"], s["beta"])
    if kind == "split":
        return mg.gemm_split(s["A"], s["B"], s["C"], s["alpha"], s["beta"], s["algo"],
                             workspace=s["ws"])
    if kind == "daxpy":
        return mg.daxpy(s["alpha"], s["x"], s["y"])
    if s["call"] == "plan":
        s["plan"].launch()
    else:
        mg.gemm_batched(s["probs"], s["dtype"], algo=s["algo"])
    return s["flat"][2]


def work(case):
    kind = case["kind"]
    if kind == "daxpy":
        return {"bytes": 24 * case["n"], "flops": 2 * case["n"]}
    if kind == "batch":
        esz = 8 if case["dtype"] == "f64" else 4
        shapes = _batch_shapes(case)
        return {"bytes": esz * sum(m * k + k * n + 2 * m * n for m, n, k in shapes),
                "flops": 2 * sum(m * n * k for m, n, k in shapes)}
    m, n, k = case["m"], case["n"], case["k"]
    esz = 4 if case.get("dtype") == "f32" else 8
    c = 2 if case["beta"] else 1
    # split precision: operations of the FP64 product it replaces
    return {"bytes": esz * (m * k + k * n + c * m * n), "flops": 2 * m * n * k}


def exact(case, seed):
    kind = case["kind"]
    if kind == "daxpy":
        x, y = _axpy_operands(case, seed)
        return y + case["alpha"] * x
    if kind == "batch":
        flat, views = _batch_operands(case, seed)
        out = flat[2].double()
        at = 0
        for A, B, C in views:
            n = C.numel()
            out[at:at + n] = (A.double() @ B.double() + C.double()).reshape(-1)
            at += -(-n // 16) * 16
        return out
    A, B, C = _operands(case, seed)
    A, B, C = A.double(), B.double(), C.double()
    if kind == "gemm":
        A = A.t().contiguous() if case["ta"] else A
        B = B.t().contiguous() if case["tb"] else B
    r = case["alpha"] * (A @ B)
    return r + case["beta"] * C if case["beta"] else r
