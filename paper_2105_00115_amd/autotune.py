"""Autotuner for the qdot launch shapes.

Single qdot, per size bucket (n < 2^16, < 2^20, < 2^24, >= 2^24): it times
the exponent scan and the accumulate pass with the library's own HIP-event
kernel timing over

* persistent-grid sizes (blocks per CU) and groups in flight per lane,
* the two forms of the accumulate pass (every candidate leaf formed in
  place, or the kept components compacted per wave),
* the number of global histogram copies the scan blocks merge into,
* the threads per block of both passes (128, 256, 512),
* the one-pass scan's grid and groups in flight,

and keeps the fastest.  Every swept shape must reproduce the reference
run's per-component classes and exponent histogram bit for bit, and the call
that is timed its counts, t, flags and bound and its value up to the rounding
of compensated FP64 sums (the classes are read from another route than the
timed one, which returns none); the one-pass value, an exact sum, must be the
same bits.  The tile structure makes that hold for every shape; the tuner
checks it for each one rather than assuming it.

Long vectors (the last bucket) count and sum in one kernel by default, behind a
sample whose grid is fixed, so there the scan's shape is timed on the
guaranteed mode, which scans the whole, and the accumulate shape on the default
mode.  The form of the accumulate pass and the threads per block choose between
the routes; the histogram copies belong to the four-kernel one, and are timed
there alone.

Solvers and batched launch, each on the benchmark workload it serves:
blocks per CU and the chunk size on the 4096 ragged instances (counts, t
and flags of every instance bit for bit), the CG gang sizing (rows per gang
block, largest gang) on the 256 CG systems launched with them, the SpMV
grid (the product bit for bit), whether the power method takes pass 1 in
its SpMV (lambda bit for bit) and the single-system CG gang.

The result is a text file that ``qdot_load_tune`` reads; ``Qdot()`` loads
``tune/<arch>_<cus>cu.txt`` next to this module when it exists.

    python -m paper_2105_00115_amd.autotune [--out PATH] [--reps 20]
"""
from __future__ import annotations

import argparse
import os
import sys
import time

# (up to 2^19 components the two-launch qdot takes one chunk per block whatever
# the shape)
BUCKET_N = [1 << 15, 3 << 18, 1 << 23, 1 << 27]
BPC = (1, 2, 4, 8, 16)
UNROLL = (1, 2, 4)
ACC_FORM = (0, 1)
HIST_COPIES = (1, 2, 4, 8)
BLOCK_THREADS = (128, 256, 512)
LONG = 1 << 24  # doubles from which the default mode guesses the classes from a sample
MARGIN = 0.02  # a non-default form must be this much faster to be kept
BATCH_BPC = (2, 3, 4)
BATCH_CHUNK = (65536, 131072, 262144)
CG_ROWS = (8192, 16384, 32768)
CG_GANG_MAX = (8, 16, 32)
SPMV_BPC = (2, 4, 8, 16)
CG_BPC = (1, 2)


def default_path(arch: str, cus: int) -> str:
    return os.path.join(os.path.dirname(os.path.abspath(__file__)), "tune",
                        f"{arch}_{cus}cu.txt")


def _time_config(h, x, y, tol, out, cfg, reps, opt=None):
    h.set_tune(-1, *cfg)
    for _ in range(3):
        h.qdot_async(x, y, tol, out, opt=opt)
    import torch
    torch.cuda.synchronize()
    h.timing_read()
    h.timing_enable(True)
    for _ in range(reps):
        h.qdot_async(x, y, tol, out, opt=opt)
    torch.cuda.synchronize()
    h.timing_enable(False)
    t = h.timing_read()
    c = t["qdot_calls"]
    return (t["scan_ms"] / c, t["cut_ms"] / c, t["acc_ms"] / c, t["fin_ms"] / c)


class ShapeChanged(RuntimeError):
    pass


FIELDS = ("count", "n_zero", "e_min", "e_max", "t", "flags", "n_bins", "bound_rel", "status")
GUARD = [0, 0, 0, 0, 1]
VALUE_TOL = 1e-14  # of sum |x_i y_i|: the order of compensated FP64 sums


def _check_same(h, x, y, tol, cfg, ref):
    """The shape cfg gives the reference classes and histogram bit for bit, and
    the routes that are timed give the reference fields and value."""
    import torch
    h.set_tune(-1, *cfg)
    cls, hist, r = h.qdot_classes(x, y, tol)
    if not (torch.equal(cls, ref["cls"]) and torch.equal(hist, ref["hist"])
            and all(r[k] == ref["res"][k] for k in FIELDS)):
        raise ShapeChanged(f"config {cfg} changed the classes or the histogram")
    for opt, want in ((None, ref["res"]), (GUARD, ref["guard"])):
        t = h.qdot(x, y, tol, opt=opt)
        if not (all(t[k] == want[k] for k in FIELDS)
                and abs(t["value"] - want["value"]) <= VALUE_TOL * ref["scale"]):
            raise ShapeChanged(f"config {cfg} changed the result (options {opt})")


def _reference(h, x, y, tol):
    cls, hist, r = h.qdot_classes(x, y, tol)
    return {"cls": cls, "hist": hist, "res": r, "guard": h.qdot(x, y, tol, opt=GUARD),
            "scale": float((x * y).abs().sum())}


def _time_routes(h, x, y, tol, out, cfg, reps, n):
    """(scan, cut, acc, fin) ms of the two-pass qdot under cfg; from
    LONG components the scan's is the guaranteed mode's."""
    t = _time_config(h, x, y, tol, out, cfg, reps)
    if n < LONG:
        return t
    return (_time_config(h, x, y, tol, out, cfg, reps, opt=GUARD)[0],) + t[1:]


def tune(reps: int = 20, seed: int = 7, tol: float = 1e-6, log=print, buckets=None):
    """Sweep the launch shapes of the buckets listed (all by default);
    returns the handle, the chosen shapes with their timings, and the number
    of shapes whose classes and histogram were compared."""
    import torch

    import paper_2105_00115_amd as q
    import workloads

    h = q.Qdot(0, load_tuned=False)
    h.reset_tune()
    dev = "cuda:0"
    out = torch.zeros(q.RESULT_BYTES, dtype=torch.uint8, device=dev)
    chosen = []
    checked = 0
    for b, n in enumerate(BUCKET_N):
        if buckets is not None and b not in buckets:
            continue
        x, y = workloads.log_uniform_pair_torch(n, seed + b, dev)
        ref = _reference(h, x, y, tol)
        d1 = h.get_tune(b)[4:6]
        # grid and groups in flight of both passes (dense form, 8 copies,
        # 256 threads per block)
        results = {}
        for bpc in BPC:
            for u in UNROLL:
                cfg = (bpc, u, bpc, u) + d1 + (0, 8, 256)
                results[cfg] = _time_routes(h, x, y, tol, out, cfg, reps, n)
                _check_same(h, x, y, tol, cfg, ref)
                checked += 1
        best_scan = min(results, key=lambda c: results[c][0])[:2]
        best_acc = min(results, key=lambda c: results[c][2])[2:4]
        mixed = best_scan + best_acc + d1 + (0, 8, 256)
        if mixed not in results:
            results[mixed] = _time_routes(h, x, y, tol, out, mixed, reps, n)
            _check_same(h, x, y, tol, mixed, ref)
            checked += 1
        best = min(results, key=lambda c: sum(results[c]))
        # accumulate form, histogram copies and threads per block at that
        # shape, by the whole call in the default mode; a shape other than the
        # default form (dense, 8 copies, 256 threads) must beat it by MARGIN on
        # a second, interleaved timing, so that noise does not pick it
        base = best[:6] + (0, 8, 256)
        cand = {}
        for af in ACC_FORM:
            for hc in HIST_COPIES:
                for nt in BLOCK_THREADS:
                    cfg = best[:6] + (af, hc, nt)
                    _check_same(h, x, y, tol, cfg, ref)
                    checked += 1
                    if (af, nt) == (0, 256) and hc != 8:
                        continue  # the copies play no part in this form
                    cand[cfg] = _time_config(h, x, y, tol, out, cfg, reps)
        challenger = min(cand, key=lambda c: sum(cand[c]))
        if challenger != base:
            tb = tc = 0.0
            for _ in range(3):
                tb += sum(_time_config(h, x, y, tol, out, base, reps))
                tc += sum(_time_config(h, x, y, tol, out, challenger, reps))
            best = challenger if tc < (1.0 - MARGIN) * tb else base
        else:
            best = base
        t = results[best] if best in results else cand[best]
        # one-pass scan (accum_mode 1): its value is an exact sum, so every
        # shape must give the same bits
        one = [0, 0, 0, 1]
        h.set_tune(-1, *best)
        ref1 = h.qdot(x, y, tol, opt=one)
        res1 = {}
        for bpc in BPC:
            for u in UNROLL:
                cfg = best[:4] + (bpc, u) + best[6:]
                res1[cfg] = _time_config(h, x, y, tol, out, cfg, reps, opt=one)
                r = q.parse_results(out)[0]
                if (r["count"], r["value"]) != (ref1["count"], ref1["value"]):
                    raise ShapeChanged(f"one-pass config {cfg} changed the result")
        best = min(res1, key=lambda c: sum(res1[c]))
        _check_same(h, x, y, tol, best, ref)
        checked += 1
        t1 = res1[best]
        log(f"bucket {b} n={n}: best {best} scan {t[0]*1e3:.1f} us cut {t[1]*1e3:.1f} us "
            f"acc {t[2]*1e3:.1f} us fin {t[3]*1e3:.1f} us; one-pass scan {t1[0]*1e3:.1f} us")
        chosen.append((b, n, best, t + (t1[0],)))
        del x, y
    return h, chosen, checked


def _time_batch(h, run, reps):
    import torch
    run()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        run()
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) / reps


def tune_batch(h, reps: int = 3, log=print):
    """Solver and batched launch shapes, each on the workload it serves:
    blocks per CU and chunk on the 4096 ragged instances of the batched
    benchmark (n = round(10^U[2,6]), tol from {1e-4, 1e-6, 1e-8}), the CG
    gang sizing on the 256 Poisson systems (sides round(2^U[5,9])) in the
    same launch, the SpMV grid on the 3D Laplacian 128^3, the single-system
    CG gang on Poisson 1024^2, and where the power method takes pass 1.
    Returns the chosen qdot_solver_tune as a tuple."""
    import numpy as np
    import torch

    import paper_2105_00115_amd as q
    import workloads

    dev = "cuda:0"
    h.set_solver_tune()
    g = workloads.rng(2025)
    sizes = np.rint(10.0 ** g.uniform(2, 6, 4096)).astype(np.int64)
    offs = np.zeros(4097, dtype=np.int64)
    np.cumsum(sizes, out=offs[1:])
    tols = np.array([1e-4, 1e-6, 1e-8])[g.integers(0, 3, 4096)]
    x, y = workloads.log_uniform_pair_torch(int(offs[-1]), 2025, dev)
    off_d = torch.from_numpy(offs).to(dev)
    tol_d = torch.from_numpy(tols).to(dev)
    out = torch.zeros(4096 * q.RESULT_BYTES, dtype=torch.uint8, device=dev)
    # one shape serves both readings: the sum of the two-pass and the
    # one-pass launch times is minimised
    modes = (None, [0, 0, 0, 1])
    refs = []
    for opt in modes:
        h.batched_async(x, y, off_d, offs, tol_d, out, opt=opt)
        torch.cuda.synchronize()
        refs.append(q.parse_results(out))
    res, per = {}, {}
    for bpc in BATCH_BPC:
        for ch in BATCH_CHUNK:
            h.set_solver_tune(batch_blocks_per_cu=bpc, batch_chunk=ch)
            per[(bpc, ch)] = []
            for opt, ref in zip(modes, refs):
                per[(bpc, ch)].append(_time_batch(
                    h, lambda: h.batched_async(x, y, off_d, offs, tol_d, out, opt=opt), reps))
                got = q.parse_results(out)
                for j, (a, r) in enumerate(zip(got, ref)):
                    if a["count"] != r["count"] or a["t"] != r["t"] or a["flags"] != r["flags"]:
                        raise ShapeChanged(f"batch shape {(bpc, ch)} changed instance {j}")
            res[(bpc, ch)] = sum(per[(bpc, ch)])
    bpc, ch = min(res, key=res.get)
    log(f"batch: best blocks/CU {bpc} chunk {ch} ({per[(bpc, ch)][0]*1e3:.3f} ms two-pass, "
        f"{per[(bpc, ch)][1]*1e3:.3f} ms one-pass for 4096 instances)")
    # CG gang sizing: the 256 systems together with the instances
    gs = workloads.rng(2026)
    sides = np.rint(2.0 ** gs.uniform(5, 9, 256)).astype(np.int64)
    mats, systems = {}, []
    rows = int((sides ** 2).sum())
    xall = torch.zeros(rows, dtype=torch.float64, device=dev)
    ball = torch.empty(rows, dtype=torch.float64, device=dev)
    ro = 0
    for k, m in enumerate(sides):
        m = int(m)
        if m not in mats:
            mats[m] = q.Csr(*workloads.poisson2d_csr(m), device=dev)
        nn = m * m
        ball[ro:ro + nn] = torch.from_numpy(workloads.normal_vector(nn, 3000 + k)).to(dev)
        systems.append((mats[m], ball[ro:ro + nn], xall[ro:ro + nn], 1e-10, 1e-8, 20000, 1))
        ro += nn
    cgo = torch.zeros(256 * q.CG_RESULT_BYTES, dtype=torch.uint8, device=dev)
    cg_res = {}
    for rpb in CG_ROWS:
        for gmax in CG_GANG_MAX:
            h.set_solver_tune(batch_blocks_per_cu=bpc, batch_chunk=ch, cg_rows_per_block=rpb,
                              cg_gang_max=gmax)
            xall.zero_()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            h.batch_run_async(x, y, off_d, offs, tol_d, out, systems, cgo)
            torch.cuda.synchronize()
            cg_res[(rpb, gmax)] = time.perf_counter() - t0
            rr = q.parse_cg_results(cgo)
            if any(r["status"] != q.OK for r in rr):
                raise RuntimeError(f"CG gang shape {(rpb, gmax)} failed")
    rpb, gmax = min(cg_res, key=cg_res.get)
    log(f"batch CG: best rows/block {rpb} gang max {gmax} ({cg_res[(rpb, gmax)]*1e3:.1f} ms "
        f"for the launch)")
    h.set_solver_tune(batch_blocks_per_cu=bpc, batch_chunk=ch, cg_rows_per_block=rpb,
                      cg_gang_max=gmax)
    del systems, mats, xall, ball, x, y
    # SpMV grid on the 3D Laplacian 128^3 (the product bit for bit the same
    # for every grid), and where the power method takes pass 1
    A = q.Csr(*workloads.laplacian3d_csr(128), device=dev)
    v = torch.from_numpy(workloads.normal_vector(A.n, 5)).to(dev)
    w = torch.empty_like(v)
    sp_res, ref_w = {}, None
    for sb in SPMV_BPC:
        h.set_solver_tune(spmv_blocks_per_cu=sb)
        sp_res[sb] = _time_batch(h, lambda: h.spmv(A, v, w), 20)
        if ref_w is None:
            ref_w = w.clone()
        elif not torch.equal(w, ref_w):
            raise ShapeChanged(f"SpMV grid {sb} changed the product")
    sb = min(sp_res, key=sp_res.get)
    log(f"SpMV: best blocks/CU {sb} ({sp_res[sb]*1e6:.1f} us)")
    x0 = workloads.unit_vector(A.n, 4)
    pm, lam = {}, {}
    for fused in (0, 1):
        h.set_solver_tune(spmv_blocks_per_cu=sb, power_scan_in_spmv=fused)
        xs = torch.from_numpy(x0).to(dev)
        h.power(A, xs, 5, 1e-6, 1, trace=False)
        xs = torch.from_numpy(x0).to(dev)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        r = h.power(A, xs, 200, 1e-6, 1, trace=False)
        pm[fused] = (time.perf_counter() - t0) / 200
        lam[fused] = r["lambda"]
    if lam[0] != lam[1]:
        raise ShapeChanged("pass 1 inside the SpMV changed the power method's lambda")
    ps = min(pm, key=pm.get)
    log(f"power: pass 1 in the SpMV {ps} ({pm[0]*1e6:.1f} / {pm[1]*1e6:.1f} us per iteration)")
    del A, v, w
    A = q.Csr(*workloads.poisson2d_csr(1024), device=dev)
    b = torch.from_numpy(workloads.normal_vector(A.n, 3)).to(dev)
    cgs = {}
    for cb in CG_BPC:
        h.set_solver_tune(spmv_blocks_per_cu=sb, power_scan_in_spmv=ps, cg_blocks_per_cu=cb)
        xx = torch.zeros(A.n, dtype=torch.float64, device=dev)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        r = h.cg(A, b, xx, 1e-10, 1e-8, 20000, 1)
        cgs[cb] = (time.perf_counter() - t0) / max(1, r["iters"])
        if r["status"] != q.OK:
            raise RuntimeError(f"CG gang of {cb} blocks per CU failed: {r}")
    cb = min(cgs, key=cgs.get)
    log(f"CG: best gang blocks/CU {cb} ({cgs[cb]*1e6:.1f} us per iteration)")
    h.set_solver_tune(spmv_blocks_per_cu=sb, power_scan_in_spmv=ps, cg_blocks_per_cu=cb)
    return h.get_solver_tune()


def write(path, chosen, arch, cus, batch=None):
    os.makedirs(os.path.dirname(path), exist_ok=True)
    with open(path, "w") as f:
        f.write(f"# qdot launch shapes for {arch} with {cus} CUs, written by "
                f"python -m paper_2105_00115_amd.autotune on {time.strftime('%Y-%m-%d')}\n")
        f.write("# bucket scan_blocks_per_cu scan_unroll acc_blocks_per_cu acc_unroll"
                " onepass_blocks_per_cu onepass_unroll acc_form hist_copies block_threads"
                "   (measured n, scan/cut/acc/fin us, one-pass scan us; cut and fin are the gap"
                " of two events where the sweep does their work; from 2^24 the scan is the"
                " guaranteed mode's)\n")
        for b, n, cfg, t in chosen:
            f.write(f"{b} {' '.join(str(c) for c in cfg)}   # n={n} "
                    f"{t[0]*1e3:.1f}/{t[1]*1e3:.1f}/{t[2]*1e3:.1f}/{t[3]*1e3:.1f}, "
                    f"{t[4]*1e3:.1f}\n")
        if batch is not None:
            f.write("# solver batch_blocks_per_cu batch_chunk cg_rows_per_block cg_gang_max"
                    " spmv_blocks_per_cu cg_blocks_per_cu power_scan_in_spmv\n")
            f.write("solver " + " ".join(str(v) for v in batch) + "\n")


def main(argv=None):
    ap = argparse.ArgumentParser()
    ap.add_argument("--out", default=None)
    ap.add_argument("--reps", type=int, default=20)
    ap.add_argument("--buckets", default=None,
                    help="comma-separated bucket indices to tune (default: all)")
    ap.add_argument("--no-batch", action="store_true", help="leave the batched shape out")
    a = ap.parse_args(argv)
    import torch

    props = torch.cuda.get_device_properties(0)
    arch = props.gcnArchName.split(":")[0]
    cus = props.multi_processor_count
    buckets = None if a.buckets is None else [int(b) for b in a.buckets.split(",")]
    log = lambda m: print(m, flush=True)  # noqa: E731
    h, chosen, checked = tune(a.reps, log=log, buckets=buckets)
    log(f"{checked} shapes gave the reference classes and histogram bit for bit")
    batch = None if a.no_batch else tune_batch(h, log=log)
    path = a.out or default_path(arch, cus)
    write(path, chosen, arch, cus, batch)
    h.load_tune(path)  # the file must load back
    print(f"wrote {path}", flush=True)


if __name__ == "__main__":
    sys.exit(main())
