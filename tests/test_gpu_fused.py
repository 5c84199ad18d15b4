"""The two-pass qdot in two launches, and in one block, at the lengths where
their dispatch and their groups end, against the oracle; and against the
four-kernel chain, which other launch shapes still take."""
import numpy as np
import pytest

import oracle
import paper_2105_00115_amd as q
import workloads

pytestmark = pytest.mark.gpu

FIELDS = ("count", "n_zero", "e_min", "e_max", "n_bins", "t", "flags", "status", "e_ref",
          "passes")
# one block: a chunk of 256 threads (1024), of 1024 threads (4096); past it
# one block per chunk up to 512 chunks, then several chunks per block; one
# copy of the counts up to 64 blocks (65536)
SIZES = [0, 1, 3, 4, 63, 65, 1023, 1024, 1025, 4095, 4096, 4097, 65535, 65537, 524288, 524289,
         1 << 20, (1 << 20) + 7]


@pytest.fixture(scope="module")
def h():
    handle = q.Qdot(0)
    yield handle
    handle.close()


def _pair(n, seed, dtype, off):
    import torch
    x, y = workloads.log_uniform_pair(n + off, seed)
    if n > 8:  # a zero product and a subnormal operand
        x[off + n // 2] = 0.0
        y[off + n // 3] = 5e-310 if dtype == np.float64 else 1e-42
    x, y = x.astype(dtype), y.astype(dtype)
    xd, yd = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(y).to("cuda:0")
    return x[off:], y[off:], xd[off:], yd[off:]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("dtype,guard,off", [(np.float64, 0, 0), (np.float64, 1, 0),
                                             (np.float64, 0, 1), (np.float32, 0, 0),
                                             (np.float32, 0, 1), (np.float32, 1, 0)])
def test_lengths(h, n, dtype, guard, off):
    x, y, xd, yd = _pair(n, 71 + n % 97, dtype, off)
    f64 = dtype == np.float64
    opt = [0, 0, 0, 0, guard]
    for tol in (1e-3, 1e-8):
        o = (oracle.qdot if f64 else oracle.qdot_f32)(x, y, tol, opt=opt)
        call = h.qdot if f64 else h.qdot_f32
        for r in (call(xd, yd, tol, opt), call(xd, yd, tol, opt)):
            for k in FIELDS:
                assert r[k] == o[k], (k, r[k], o[k])
            assert abs(r["value"] - o["value"]) <= 1e-13 * oracle.abs_dot(
                x.astype(np.float64), y.astype(np.float64))


@pytest.mark.parametrize("n", [700, 3000, 30000, 200000, 600000])
@pytest.mark.parametrize("opt", [[0, 0, 0, 0, 0], [1, 1, 0, 0, 0], [0, 0, 1, 0, 0],
                                 [0, 0, 0, 0, 1], [0, 1, 1, 0, 1]])
def test_same_as_four_kernel_chain(h, n, opt):
    """Every form of the options, on cancelling sums (which the guaranteed
    mode selects again): the classes, counts and leaves are the chain's, the
    compensated FP64 sums differ by their error terms' rounding at most."""
    import torch
    x, y = workloads.cancelling_pair(n, n, 3e-4)
    xd, yd = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(y).to("cuda:0")
    with q.Qdot(0) as other:
        other.set_tune(-1, 2, 1, 2, 1, block_threads=128)
        for tol in (1e-2, 1e-5):
            r, c = h.qdot(xd, yd, tol, opt), other.qdot(xd, yd, tol, opt)
            for k in FIELDS:
                assert r[k] == c[k], (k, r[k], c[k])
            assert r["bound_rel"] == c["bound_rel"]
            assert abs(r["value"] - c["value"]) <= 4e-16 * oracle.abs_dot(x, y)


@pytest.mark.parametrize("n", [1000, 4000, 100000])
def test_error_results_leave_the_workspace_clean(h, n):
    import torch
    x, y, xd, yd = _pair(n, 5, np.float64, 0)
    bad = xd.clone()
    bad[n - 1] = float("inf")
    ref = h.qdot(xd, yd, 1e-6)
    e = h.qdot(bad, yd, 1e-6)
    assert e["status"] == q.E_NONFINITE and np.isnan(e["value"]) and e["count"] == [0] * 4
    z = h.qdot(torch.zeros_like(xd), yd, 1e-6, [0, 0, 0, 0, 1])
    assert z["value"] == 0.0 and z["n_zero"] == n and z["flags"] & q.F_GUARANTEED
    assert h.qdot(xd, yd, 1e-6) == ref


@pytest.mark.parametrize("m", [1, 5, 16, 64, 82])
@pytest.mark.parametrize("opt", [[0, 0, 0, 0, 0], [1, 0, 1, 0, 0], [0, 0, 0, 0, 1]])
def test_power_pair(m, opt):
    """The pair of inner products of a power step in two launches, against
    the four-kernel chain of the other launch shapes: every field but the
    compensated sums' last bits."""
    import torch
    A = q.Csr(*workloads.laplacian3d_csr(m))
    x0 = torch.from_numpy(workloads.unit_vector(A.n, m + 2)).to("cuda:0")
    res = []
    for nt in (256, 128):
        with q.Qdot(0) as hh:
            hh.set_tune(-1, 2, 1, 2, 1, block_threads=nt)
            res.append(hh.power(A, x0.clone(), 6, 1e-6, 1, opt=opt, results=True))
    for a, b in zip(*(r["results"] for r in res)):
        for k in FIELDS:
            assert a[k] == b[k], (k, a[k], b[k])
        # products of one sign (w . w) or nearly cancelling ones (x . w): the
        # sum of |x_i w_i| is at most sqrt(x.x) sqrt(w.w) <= 12
        assert abs(a["value"] - b["value"]) <= 12 * 1e-13


@pytest.mark.parametrize("count", [1, 3, 767, 769, 1600])
@pytest.mark.parametrize("guard", [0, 1])
def test_small_instances_spread_over_blocks(h, count, guard):
    """Runs of small instances at one instance per block, at one more than
    the resident blocks and at two per block, with lengths around a chunk and
    a group: each instance against the oracle."""
    import torch
    lens = [(0, 1, 63, 1024, 1025, 2047, 2048, 2049, 300)[i % 9] for i in range(count)]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(off[-1])
    x, y = workloads.log_uniform_pair(n + 1, 40 + count)
    x, y = x[:n], y[:n]
    if n:
        x[n // 2] = 0.0
    tols = [(1e-4, 1e-6, 1e-8)[i % 3] for i in range(count)]
    xd, yd = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(y).to("cuda:0")
    opt = [0, 0, 0, 0, guard]
    for _ in range(2):
        res = h.batched(xd, yd, off, tols, opt)
        for j, r in enumerate(res):
            a, b = x[off[j]:off[j + 1]], y[off[j]:off[j + 1]]
            o = oracle.qdot(a, b, tols[j], opt=opt)
            for k in ("count", "n_zero", "e_min", "e_max", "n_bins", "t", "flags", "status"):
                assert r[k] == o[k], (j, k, r[k], o[k])
            assert abs(r["value"] - o["value"]) <= 1e-13 * oracle.abs_dot(a, b)


@pytest.mark.parametrize("sides", [[1], [33], [32, 40, 200], [32] * 40 + [181], [100] * 70,
                                   [300, 300, 299]])
def test_gangs_shared_out(h, sides):
    """Batches whose gangs would leave resident blocks idle get larger ones:
    rows split at every chunk, a gang of one block, gangs at the bound of 64,
    and a batch that fills the chip at the tuned shape.  Each system takes the
    iteration count and the solution of the single-system solve, whose gang
    has another shape (every inner product is the same but for FP64 error
    terms, so 40 iterations stay far above the tolerance's 1e-9)."""
    import torch
    systems = []
    for i, m in enumerate(sides):
        A = q.Csr(*workloads.poisson2d_csr(m))
        b = torch.from_numpy(workloads.normal_vector(A.n, 60 + i)).to("cuda:0")
        systems.append((A, b, torch.zeros_like(b), 1e-8, 1e-8, 40, 1))
    res = h.cg_batched(systems)
    for (A, b, x, *_), r in list(zip(systems, res))[::max(1, len(sides) // 4)]:
        xs = torch.zeros_like(b)
        one = h.cg(A, b, xs, 1e-8, 1e-8, 40, 1)
        assert (r["iters"], r["status"]) == (one["iters"], one["status"])
        assert float((x - xs).norm()) <= 1e-9 * float(xs.norm())


def _shuffled_rows_csr(n, long_rows, seed):
    """SPD, diagonally dominant: random_spd_csr plus rows of several hundred
    entries at the places given (symmetric, so their columns grow too)."""
    rp, col, val = workloads.random_spd_csr(n, 2, seed)
    g = workloads.rng(seed + 1)
    i = np.repeat(np.arange(n), np.diff(rp))
    rows, cols, vals = [i], [col.astype(np.int64)], [val]
    for r in long_rows:
        c = g.choice(n, 300, replace=False)
        c = c[c != r]
        v = -g.uniform(1e-4, 1e-3, c.shape[0])
        rows += [np.full(c.shape[0], r), c]
        cols += [c, np.full(c.shape[0], r)]
        vals += [v, v]
    import scipy.sparse as sp
    A = sp.coo_matrix((np.concatenate(vals), (np.concatenate(rows), np.concatenate(cols))),
                      shape=(n, n)).tocsr()
    A = A + sp.diags(np.asarray(abs(A).sum(axis=1)).ravel())
    A.sort_indices()
    return A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data


@pytest.mark.parametrize("n,long_rows", [(1, ()), (1023, ()), (1025, (7,)), (5000, (0, 1023, 4999)),
                                         (40000, (5, 20000, 39999)), (270000, (12, 1030))])
@pytest.mark.parametrize("opt", [[0, 0, 0, 0, 0], [0, 0, 0, 0, 1], [0, 0, 0, 1, 0]])
def test_cg_resident_rows(h, n, long_rows, opt):
    """Rows in LDS, the row ahead in registers, rows after them and rows past
    the eight gathered at once, over slices of one block up to several rows
    per thread: the iterate of each step against the oracle's.  A step's
    error is the tolerance's (1e-10 of each inner product) and the FP64
    rounding's, and these systems have condition numbers near 2, so after 12
    steps the iterates agree to far below 1e-8."""
    import torch
    rp, col, val = (workloads.random_spd_csr(n, 3, 5) if not long_rows
                    else _shuffled_rows_csr(n, long_rows, 5))
    if n == 1:
        rp, col, val = np.array([0, 1], np.int32), np.zeros(1, np.int32), np.full(1, 3.0)
    b = workloads.normal_vector(n, 9)
    A = q.Csr(rp, col, val)
    bd = torch.from_numpy(b).to("cuda:0")
    x = torch.zeros_like(bd)
    r = h.cg(A, bd, x, 1e-300, 1e-10, 12, 1, opt)
    o = oracle.cg(rp, col, val, b, 1e-300, 1e-10, 12, 1, opt=opt)
    ox = o["x"]
    assert abs(r["iters"] - o["iters"]) <= (0 if n > 1 else 12)
    assert np.linalg.norm(x.cpu().numpy() - ox) <= 1e-8 * np.linalg.norm(ox)


def _long_pair(n, law, seed):
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    if law == "loguniform":
        return workloads.log_uniform_pair_torch(n, seed)
    if law == "familyA":
        return workloads.paper_dist_torch(n, 13, seed, "A")
    x = torch.randn(n, generator=g, dtype=torch.float64, device="cuda:0")
    y = torch.randn(n, generator=g, dtype=torch.float64, device="cuda:0")
    if law == "late":  # its second half 40 binades up: a sample's tail looks ended, but is not
        x[n // 2 + 12345:n // 2 + 12500] *= 2.0 ** 40
    if law == "sample only":  # the largest products lie in the sample's runs alone
        x.view(-1)[:4096] *= 2.0 ** 40
    if law == "constant":
        return torch.ones_like(x), torch.full_like(x, 1.5)
    if law == "zeros":
        x.zero_()
    if law == "inf":
        x[n - 1] = float("inf")
    return x, y


@pytest.mark.parametrize("n,off", [(1 << 24, 0), ((1 << 24) + 1, 0), ((1 << 24) + 4097, 1),
                                   (31_000_003, 0), ((1 << 25) - 5, 0)])
@pytest.mark.parametrize("law", ["loguniform", "familyA", "normal", "late", "sample only",
                                 "constant", "zeros", "inf"])
def test_long_vectors_by_guess(h, n, off, law):
    """Sums by guessed classes: guesses that stand, that are not used, and that
    are wrong (the sample never sees the largest exponents), against the
    four-kernel chain: every integer field, and the value up to the FP64
    sums' error terms (2 units in the last place of sum |x_i y_i|)."""
    import torch
    x, y = _long_pair(n + off, law, 11)
    x, y = x[off:], y[off:]
    scale = float((x * y).abs().sum()) if law != "inf" else 1.0
    with q.Qdot(0) as other:
        other.set_tune(-1, 2, 1, 2, 1, block_threads=128)
        for tol, opt in ((1e-3, None), (1e-6, None), (1e-10, [1, 1, 1, 0])):
            c = other.qdot(x, y, tol, opt)
            for r in (h.qdot(x, y, tol, opt), h.qdot(x, y, tol, opt)):
                for k in FIELDS:
                    assert r[k] == c[k], (law, tol, k, r[k], c[k])
                assert r["bound_rel"] == c["bound_rel"]
                if law == "inf":
                    assert np.isnan(r["value"])
                else:
                    assert abs(r["value"] - c["value"]) <= 4.5e-16 * scale
        if law in ("loguniform", "normal", "late"):
            xf, yf = torch.cat([x, x])[:1 << 25].float(), torch.cat([y, y])[:1 << 25].float()
            xf, yf = torch.cat([xf, xf[:3000]]), torch.cat([yf, yf[:3000]])
            c = other.qdot_f32(xf, yf, 1e-6)
            # the chain's float grouping is this path's own (the threads knob is
            # for doubles), so only the routes differ
            for r in (h.qdot_f32(xf, yf, 1e-6), h.qdot_f32(xf, yf, 1e-6)):
                for k in FIELDS:
                    assert r[k] == c[k], (law, k, r[k], c[k])
                assert abs(r["value"] - c["value"]) <= 4.5e-16 * float(
                    (xf.double() * yf.double()).abs().sum())


@pytest.mark.parametrize("n", [0, 3, 1000, 4096, 4097, 100001, (1 << 24) + 5])
@pytest.mark.parametrize("dtype,opt", [(np.float64, [0, 0, 0, 0, 0]), (np.float64, [0, 0, 0, 0, 1]),
                                       (np.float64, [0, 0, 0, 1, 0]), (np.float32, [0, 0, 0, 0, 0])])
def test_synchronous_result_is_the_asynchronous_one(h, n, dtype, opt):
    """The synchronous call's result, which some paths store into host memory
    and others have copied there, is the asynchronous call's, byte for byte:
    also after a result of another length, and of an error."""
    import torch
    *_, xd, yd = _pair(n, 5 + n, dtype, 0)
    f64 = dtype == np.float64
    sync, enqueue = (h.qdot, h.qdot_async) if f64 else (h.qdot_f32, h.qdot_f32_async)
    bad = xd.clone()
    if n:
        bad[n // 2] = float("nan")
    out = torch.zeros(q.RESULT_BYTES, dtype=torch.uint8, device="cuda:0")
    for v in (xd, bad, xd):
        enqueue(v, yd, 1e-5, out, opt)
        torch.cuda.synchronize()
        want = q.QdotResult.from_buffer_copy(out.cpu().numpy().tobytes()).as_dict()
        r = sync(v, yd, 1e-5, opt)
        assert repr(r) == repr(want)
