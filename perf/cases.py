"""The calls that a program using this library makes, for timing and for
comparing results.

listed() names them; draw(rng) gives one more of the same ranges;
prepare(case, seed) makes what the program holds before the call, run(state)
makes the call, work(case) says what it cannot do without, exact(case, seed)
gives the same outputs from plain 64-bit torch.

A case is one of five kinds:
  single  one qdot of two vectors (two-pass, one-pass or guaranteed mode,
          double or single precision)
  batch   ragged qdot instances in one launch
  cg      conjugate gradient on the 2D 5-point Poisson operator
  cgs     many such systems in one launch
  power   the power method on the 3D 7-point Laplacian
"""
import functools
import math

import torch

import paper_2105_00115_amd as q

DEV = "cuda:0"


def listed():
    return [
        # a scalar that the host needs at once (a convergence test on a short
        # vector): the synchronous call, nothing but latency
        {"name": "sync 1e3", "kind": "single", "n": 1000, "law": "loguniform", "tol": 1e-6,
         "dtype": "f64", "mode": "two-pass", "sync": True},
        # the ordinary small call, its result left on the device
        {"name": "1e5", "kind": "single", "n": 100_000, "law": "loguniform", "tol": 1e-6,
         "dtype": "f64", "mode": "two-pass", "sync": False},
        # a certified product of an odd length, components of one size
        {"name": "guaranteed 1e6+3", "kind": "single", "n": 1_000_003, "law": "normal",
         "tol": 1e-8, "dtype": "f64", "mode": "guaranteed", "sync": False},
        # the second family of the error-bound study at its third size
        {"name": "family B 1e7", "kind": "single", "n": 10_000_000, "law": "familyB9",
         "tol": 1e-4, "dtype": "f64", "mode": "two-pass", "sync": False},
        # the benchmark's vectors: 1 GiB each
        {"name": "2^27", "kind": "single", "n": 1 << 27, "law": "loguniform", "tol": 1e-6,
         "dtype": "f64", "mode": "two-pass", "sync": False},
        # the same in the mode that reads them once
        {"name": "one-pass 2^27", "kind": "single", "n": 1 << 27, "law": "loguniform",
         "tol": 1e-6, "dtype": "f64", "mode": "one-pass", "sync": False},
        # single-precision vectors of an odd length
        {"name": "f32 5e7+17", "kind": "single", "n": 50_000_017, "law": "loguniform",
         "tol": 1e-6, "dtype": "f32", "mode": "two-pass", "sync": False},
        # ragged instances, as many and as long as the benchmark's
        {"name": "batch 4096", "kind": "batch", "count": 4096, "n_lo": 100, "n_hi": 1_000_000,
         "mode": "two-pass"},
        # a few hundred short ones: the launch's fixed costs
        {"name": "batch 256 short", "kind": "batch", "count": 256, "n_lo": 100, "n_hi": 10_000,
         "mode": "two-pass"},
        # the solver on the benchmark's grid, some iterations of it
        {"name": "cg 1024", "kind": "cg", "side": 1024, "iters": 60, "mode": "two-pass"},
        # many small and middling systems together
        {"name": "cg batch 24", "kind": "cgs", "count": 24, "side_lo": 32, "side_hi": 512,
         "iters": 60},
        # the eigenvalue solver on the benchmark's grid, some iterations of it
        {"name": "power 128", "kind": "power", "side": 128, "iters": 40, "mode": "two-pass"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["single"] * 6 + ["batch"] * 2 + ["cg", "cgs", "power"])
    if kind == "single":
        dtype = rng.choice(["f64", "f64", "f32"])
        n = _log_int(rng, 1000, 1 << 27)
        return {"kind": kind, "n": n,
                "law": rng.choice(["loguniform", "normal", "familyA13", "familyB5",
                                   "familyB9", "familyB13"]),
                "tol": rng.choice([1e-3, 1e-4, 1e-6, 1e-8, 1e-10]), "dtype": dtype,
                "mode": rng.choice(["two-pass", "two-pass", "one-pass", "guaranteed"]
                                   if dtype == "f64" else ["two-pass", "two-pass", "one-pass"]),
                "sync": n < 20000 and rng.random() < 0.5}
    if kind == "batch":
        lo = _log_int(rng, 20, 1000)
        hi = _log_int(rng, 4 * lo, 1_000_000)
        most = int(4e8 / ((hi - lo) / math.log(hi / lo)))
        return {"kind": kind, "count": min(_log_int(rng, 64, 4096), most), "n_lo": lo,
                "n_hi": hi, "mode": rng.choice(["two-pass", "two-pass", "one-pass"])}
    if kind == "cg":
        return {"kind": kind, "side": _log_int(rng, 64, 1024), "iters": rng.randint(30, 60),
                "mode": rng.choice(["two-pass", "two-pass", "one-pass", "guaranteed"])}
    if kind == "cgs":
        return {"kind": kind, "count": rng.randint(8, 24), "side_lo": 32,
                "side_hi": _log_int(rng, 128, 512), "iters": rng.randint(30, 60)}
    return {"kind": kind, "side": _log_int(rng, 24, 128), "iters": rng.randint(20, 40),
            "mode": rng.choice(["two-pass", "two-pass", "one-pass"])}


# ---- inputs ------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _vector(n, law, g):
    """One vector of the law: +-10**U[-20, 20], standard normal, or the
    families s * 2**p, s ~ U[0.5, 1), p uniform (A) or normal (B) and
    rounded, with the width after the letter."""
    if law == "normal":
        return torch.randn(n, generator=g, dtype=torch.float64, device=DEV)
    if law == "loguniform":
        v = torch.rand(n, generator=g, dtype=torch.float64, device=DEV)
        v = torch.pow(10.0, v.mul_(40.0).sub_(20.0))
        s = torch.randint(0, 2, (n,), generator=g, device=DEV, dtype=torch.int8)
        return v.mul_(1.0 - 2.0 * s.to(torch.float64))
    t = float(law[7:])
    s = torch.rand(n, generator=g, dtype=torch.float64, device=DEV).mul_(0.5).add_(0.5)
    if law.startswith("familyA"):
        p = torch.rand(n, generator=g, dtype=torch.float64, device=DEV).mul_(t).sub_(0.5 * t)
    else:
        p = torch.randn(n, generator=g, dtype=torch.float64, device=DEV).mul_(0.5 * t)
    return torch.ldexp(s, torch.round(p))


def _stencil(side, dims):
    """CSR of the Dirichlet Laplacian on a side**dims grid (diagonal 2 dims,
    neighbours -1, columns ascending), built on the device."""
    n = side ** dims
    idx = torch.arange(n, device=DEV, dtype=torch.int64)
    steps = [side ** a for a in reversed(range(dims))]      # slowest axis first
    cols, keep = [], []
    for st in steps:
        cols.append(idx - st)
        keep.append((idx // st) % side > 0)
    cols.append(idx)
    keep.append(torch.ones(n, dtype=torch.bool, device=DEV))
    for st in reversed(steps):
        cols.append(idx + st)
        keep.append((idx // st) % side < side - 1)
    keep = torch.stack(keep, 1)
    col = torch.stack(cols, 1)[keep].to(torch.int32)
    val = torch.full((2 * dims + 1,), -1.0, dtype=torch.float64, device=DEV)
    val[dims] = 2.0 * dims
    val = val.expand(n, -1)[keep].contiguous()
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = keep.sum(1).cumsum(0)
    return q.Csr(rowptr.to(torch.int32), col, val, DEV)


def _lengths(case, seed):
    g = torch.Generator()
    g.manual_seed(int(seed))
    u = torch.rand(case["count"], generator=g, dtype=torch.float64)
    lo, hi = math.log(case["n_lo"]), math.log(case["n_hi"])
    return torch.exp(lo + (hi - lo) * u).round().to(torch.int64)


def _sides(case):
    """The systems' grid sides, evenly spread over the logarithm of the range."""
    lo, ratio = case["side_lo"], case["side_hi"] / case["side_lo"]
    return [round(lo * ratio ** (i / (case["count"] - 1))) for i in range(case["count"])]


@functools.cache
def _handle():
    """The handle that a program keeps."""
    return q.Qdot(0)


def _options(mode):
    return {"two-pass": None, "one-pass": q.QdotOptions(accum_mode=1),
            "guaranteed": q.QdotOptions(guard_mode=1)}[mode]


def _result_views(buf, count):
    """The fields of `count` result records in a byte tensor, as views."""
    rec = buf.view(count, q.RESULT_BYTES)

    def field(name, dtype, k=1):
        at = getattr(q.QdotResult, name).offset
        size = torch.empty(0, dtype=dtype).element_size()
        return rec[:, at:at + k * size].view(dtype)

    out = {"value": field("value", torch.float64), "count": field("count", torch.int64, 4),
           "n_zero": field("n_zero", torch.int64), "part": field("part", torch.float64, 3),
           "bound": field("bound_rel", torch.float64, 2),
           "lower": field("lower", torch.float64)}
    for name in ("e_min", "e_max", "n_bins", "t", "flags", "status", "e_ref", "passes"):
        out[name] = field(name, torch.int32)
    return out


RTOL, QTOL_CG, QTOL_POWER = 1e-10, 1e-8, 1e-6
BATCH_TOLS = (1e-4, 1e-6, 1e-8)


def prepare(case, seed):
    g = _gen(seed)
    s = {"case": case, "h": _handle()}
    kind = case["kind"]
    if kind == "single":
        dtype = torch.float32 if case["dtype"] == "f32" else torch.float64
        s["x"] = _vector(case["n"], case["law"], g).to(dtype)
        s["y"] = _vector(case["n"], case["law"], g).to(dtype)
        s["opt"] = _options(case["mode"])
        s["buf"] = torch.zeros(q.RESULT_BYTES, dtype=torch.uint8, device=DEV)
        s["out"] = _result_views(s["buf"], 1)
    elif kind == "batch":
        lens = _lengths(case, seed)
        off = torch.zeros(case["count"] + 1, dtype=torch.int64)
        off[1:] = lens.cumsum(0)
        total = int(off[-1])
        s["x"] = _vector(total, "loguniform", g)
        s["y"] = _vector(total, "loguniform", g)
        s["host_off"], s["off"] = off.numpy(), off.to(DEV)
        pick = torch.randint(0, 3, (case["count"],), generator=g, device=DEV)
        s["tol"] = torch.tensor(BATCH_TOLS, dtype=torch.float64, device=DEV)[pick]
        s["opt"] = _options(case["mode"])
        s["buf"] = torch.zeros(case["count"] * q.RESULT_BYTES, dtype=torch.uint8, device=DEV)
        s["out"] = _result_views(s["buf"], case["count"])
        s["h"].batch_plan(s["host_off"], [], s["opt"])
    elif kind == "cg":
        s["A"] = _stencil(case["side"], 2)
        s["b"] = torch.randn(s["A"].n, generator=g, dtype=torch.float64, device=DEV)
        s["x"] = torch.zeros_like(s["b"])
        s["opt"] = _options(case["mode"])
    elif kind == "cgs":
        s["systems"] = []
        for side in _sides(case):
            A = _stencil(side, 2)
            b = torch.randn(A.n, generator=g, dtype=torch.float64, device=DEV)
            s["systems"].append((A, b, torch.zeros_like(b), RTOL, QTOL_CG, case["iters"], 1))
    else:
        s["A"] = _stencil(case["side"], 3)
        v = torch.randn(s["A"].n, generator=g, dtype=torch.float64, device=DEV)
        s["start"] = v / v.norm()
        s["x"] = torch.empty_like(v)
        s["opt"] = _options(case["mode"])
    return s


def run(s):
    case, h = s["case"], s["h"]
    kind = case["kind"]
    if kind == "single":
        f32 = case["dtype"] == "f32"
        if case["sync"]:
            return (h.qdot_f32 if f32 else h.qdot)(s["x"], s["y"], case["tol"], s["opt"])
        (h.qdot_f32_async if f32 else h.qdot_async)(s["x"], s["y"], case["tol"], s["buf"],
                                                    s["opt"])
        return s["out"]
    if kind == "batch":
        h.batched_async(s["x"], s["y"], s["off"], s["host_off"], s["tol"], s["buf"], s["opt"])
        return s["out"]
    if kind == "cg":
        s["x"].zero_()
        r = h.cg(s["A"], s["b"], s["x"], RTOL, QTOL_CG, case["iters"], 1, s["opt"])
        return {"x": s["x"], **r}
    if kind == "cgs":
        for _, _, x, *_ in s["systems"]:
            x.zero_()
        r = h.cg_batched(s["systems"])
        return {"x": torch.cat([t[2] for t in s["systems"]]),
                "iters": torch.tensor([d["iters"] for d in r]),
                "status": torch.tensor([d["status"] for d in r]),
                "relres": torch.tensor([d["relres_est"] for d in r], dtype=torch.float64)}
    s["x"].copy_(s["start"])
    r = h.power(s["A"], s["x"], case["iters"], QTOL_POWER, 1, s["opt"])
    return {"x": s["x"], "lambda": r["lambda"], "trace": r["trace"], "status": r["status"]}


# ---- what a pass cannot do without ---------------------------------------------
def _nnz(side, dims):
    return (2 * dims + 1) * side ** dims - 2 * dims * side ** (dims - 1)


def _cg_work(side, iters):
    # an iteration reads the matrix once, and reads and writes x, r and p
    n, nnz = side * side, _nnz(side, 2)
    return iters * (12 * nnz + 4 * n + 48 * n), iters * (2 * nnz + 10 * n)


def work(case):
    kind = case["kind"]
    if kind == "single":
        size = 4 if case["dtype"] == "f32" else 8
        return {"bytes": 2 * size * case["n"] + q.RESULT_BYTES, "flops": 2 * case["n"]}
    if kind == "batch":
        lo, hi = case["n_lo"], case["n_hi"]
        n = case["count"] * (hi - lo) / math.log(hi / lo)   # the mean length times the count
        return {"bytes": 16 * n + q.RESULT_BYTES * case["count"], "flops": 2 * n}
    if kind == "cg":
        b, f = _cg_work(case["side"], case["iters"])
        return {"bytes": b, "flops": f}
    if kind == "cgs":
        each = [_cg_work(side, case["iters"]) for side in _sides(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    # an iteration reads the matrix and x once and writes x
    n, nnz = case["side"] ** 3, _nnz(case["side"], 3)
    return {"bytes": case["iters"] * (12 * nnz + 4 * n + 16 * n),
            "flops": case["iters"] * (2 * nnz + 5 * n)}


# ---- the same outputs from plain 64-bit torch -------------------------------------
RESULT_NAMES = ("value", "count", "n_zero", "part", "bound", "lower", "e_min", "e_max",
                "n_bins", "t", "flags", "status", "e_ref", "passes")


def _laplace(u):
    """The Dirichlet Laplacian on the grid u."""
    y = 2.0 * u.dim() * u
    for a in range(u.dim()):
        y.narrow(a, 1, u.shape[a] - 1).sub_(u.narrow(a, 0, u.shape[a] - 1))
        y.narrow(a, 0, u.shape[a] - 1).sub_(u.narrow(a, 1, u.shape[a] - 1))
    return y


def _cg(b, iters):
    """(x, ||r||/||b||) after `iters` steps, or at the tolerance."""
    x, r, p = torch.zeros_like(b), b.clone(), b.clone()
    c = (r * r).sum()
    b2 = c.clone()
    for _ in range(iters):
        if float(c) <= RTOL * RTOL * float(b2):
            break
        w = _laplace(p)
        alpha = c / (p * w).sum()
        x += alpha * p
        r -= alpha * w
        c, c0 = (r * r).sum(), c
        p = r + (c / c0) * p
    return x.reshape(-1), float((c / b2).sqrt())


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    if kind == "single":
        if case["sync"]:
            none = {k: None for k in q.QdotResult().as_dict()}
            none["count"], none["part"] = [None] * 4, [None] * 3
            return {**none, "value": float((s["x"].double() * s["y"].double()).sum())}
        v = torch.zeros(1, 1, dtype=torch.float64, device=DEV)
        for i in range(0, case["n"], 1 << 24):
            v += (s["x"][i:i + (1 << 24)].double() * s["y"][i:i + (1 << 24)].double()).sum()
        return {**dict.fromkeys(RESULT_NAMES), "value": v}
    if kind == "batch":
        v = [(s["x"][a:b] * s["y"][a:b]).sum()
             for a, b in zip(s["host_off"][:-1].tolist(), s["host_off"][1:].tolist())]
        return {**dict.fromkeys(RESULT_NAMES), "value": torch.stack(v).reshape(-1, 1)}
    if kind == "cg":
        x, _ = _cg(s["b"].view(case["side"], case["side"]), case["iters"])
        return {"x": x, "status": None, "iters": None, "relres_est": None, "relres_true": None}
    if kind == "cgs":
        xs = [_cg(b.view(math.isqrt(A.n), -1), case["iters"])[0]
              for A, b, *_ in s["systems"]]
        return {"x": torch.cat(xs), "iters": None, "status": None, "relres": None}
    u = s["start"].view((case["side"],) * 3).clone()
    trace = []
    for _ in range(case["iters"]):
        w = _laplace(u)
        trace.append((u * w).sum())
        u = w / (w * w).sum().sqrt()
    return {"x": u.reshape(-1), "lambda": float(trace[-1]), "trace": torch.stack(trace),
            "status": None}
