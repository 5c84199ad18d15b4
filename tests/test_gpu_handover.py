"""What blocks and launches hand to one another: verdicts, published values and
clean workspaces, over calls that take different paths on one handle."""
import numpy as np
import pytest

import oracle
import paper_2105_00115_amd as q
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    handle = q.Qdot(0)
    yield handle
    handle.close()


def test_guess_verdicts_do_not_outlive_their_call(h):
    """Calls on one handle whose guess stands, is not used and is wrong, in
    turn and without a wait between them: every result is its first one, byte
    for byte (each of them is checked against the chain elsewhere)."""
    import torch
    n = 1 << 24
    xs = workloads.log_uniform_pair_torch(n, 3)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(4)
    normal = tuple(torch.randn(n, generator=g, dtype=torch.float64, device="cuda:0")
                   for _ in range(2))
    late = (xs[0].clone(), xs[1])
    late[0][n // 2 + 12345:n // 2 + 12500] *= 2.0 ** 300
    pairs = (xs, normal, late)
    out = torch.zeros((20, 3, q.RESULT_BYTES), dtype=torch.uint8, device="cuda:0")
    for row in out:
        for (x, y), slot in zip(pairs, row):
            h.qdot_async(x, y, 1e-6, slot)
    res = out.cpu().numpy()
    first = [q.parse_results(res[0, k].tobytes())[0] for k in range(3)]
    for (x, y), r in zip(pairs, first):
        assert r["status"] == q.OK and sum(r["count"]) == n and r["n_bins"] > 0
        assert r["value"] != 0.0
    for row in res[1:]:
        assert np.array_equal(row, res[0])


@pytest.mark.parametrize("blocks", [1, 2, 63, 64, 65, 128, 129, 256])
def test_fp64_dots_in_a_row(h, blocks):
    """CG with the FP64 dot, whose inner products follow one another without a
    barrier between, in gangs around the 64 blocks that one wave of block 0
    waits for: the oracle's iteration count and solution.  Each step's error is
    FP64 rounding times a condition number below 20, so the iterates
    agree to far below 1e-9."""
    import torch
    n = 1024 * blocks - 3
    rp, col, val = workloads.random_spd_csr(n, 3, 5)
    A = q.Csr(rp, col, val)
    b = workloads.normal_vector(n, 9)
    o = oracle.cg(rp, col, val, b, 1e-9, 1e-10, 40, 0)
    bd = torch.from_numpy(b).to("cuda:0")
    for _ in range(3):
        x = torch.zeros_like(bd)
        r = h.cg(A, bd, x, 1e-9, 1e-10, 40, 0)
        assert (r["status"], r["iters"]) == (o["status"], o["iters"])
        assert np.linalg.norm(x.cpu().numpy() - o["x"]) <= 1e-9 * np.linalg.norm(o["x"])


@pytest.mark.parametrize("gang_max", [64, 65, 200])
def test_fp64_dots_in_a_row_batched(gang_max):
    """The same in the batched launch, whose blocks have 256 threads."""
    import torch
    with q.Qdot(0) as hh:
        hh.set_solver_tune(cg_rows_per_block=1024, cg_gang_max=gang_max)
        systems, want = [], []
        for m in (gang_max, 3):
            n = 1024 * m - 5
            rp, col, val = workloads.random_spd_csr(n, 3, 7)
            b = workloads.normal_vector(n, 3)
            bd = torch.from_numpy(b).to("cuda:0")
            systems.append((q.Csr(rp, col, val), bd, torch.zeros_like(bd), 1e-9, 1e-10, 40, 0))
            want.append(oracle.cg(rp, col, val, b, 1e-9, 1e-10, 40, 0))
        for _ in range(3):
            for s in systems:
                s[2].zero_()
            for (_, _, x, *_), r, o in zip(systems, hh.cg_batched(systems), want):
                assert (r["status"], r["iters"]) == (o["status"], o["iters"])
                assert np.linalg.norm(x.cpu().numpy() - o["x"]) <= 1e-9 * np.linalg.norm(o["x"])


@pytest.mark.parametrize("guard", [0, 1])
def test_blocks_of_a_gang_that_gave_up_go_on_clean(guard, monkeypatch):
    """A gang whose waits are given up at once (a spin limit of none, and one
    block held up by a row as long as the matrix) reports it, and its blocks
    then take qdot instances of the same launch: their results are those of a
    launch without the system, byte for byte.  The next launch on the same
    handle starts clean."""
    import torch
    n, gang = 65 * 1024, 65
    rp, col, val = workloads.random_spd_csr(n, 2, 5)
    r = 40 * 1024 + 7  # the long row, in the slice of block 40
    rp, col, val = rp.astype(np.int64), col.astype(np.int64), val.astype(np.float64)
    full = np.arange(n)
    head, tail = slice(0, rp[r]), slice(rp[r + 1], None)
    col2 = np.concatenate([col[head], full, col[tail]]).astype(np.int32)
    val2 = np.concatenate([val[head], np.full(n, 1e-6), val[tail]])
    rp2 = rp.copy()
    rp2[r + 1:] += n - (rp[r + 1] - rp[r])
    A = q.Csr(rp2.astype(np.int32), col2, val2)
    b = torch.from_numpy(workloads.normal_vector(n, 2)).to("cuda:0")
    lens = [100000 + 37 * (i % 50) for i in range(3000)] + [400000, 300001]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    # of the size of the system's residuals, so that counts left behind show
    g = torch.Generator(device="cuda:0")
    g.manual_seed(6)
    x, y = (torch.randn(int(off[-1]), generator=g, dtype=torch.float64, device="cuda:0")
            for _ in range(2))
    off_d = torch.from_numpy(off).to("cuda:0")
    tols = torch.full((len(lens),), 1e-6, dtype=torch.float64, device="cuda:0")
    opt = [0, 0, 0, 0, guard]
    res = [torch.zeros(len(lens) * q.RESULT_BYTES, dtype=torch.uint8, device="cuda:0")
           for _ in range(2)]
    with q.Qdot(0) as plain:
        plain.batched_async(x, y, off_d, off, tols, res[0], opt=opt)
        torch.cuda.synchronize()
    monkeypatch.setenv("QDOT_SPIN_LIMIT", "0")
    cg_out = torch.zeros(q.CG_RESULT_BYTES, dtype=torch.uint8, device="cuda:0")
    with q.Qdot(0) as hh:
        hh.set_solver_tune(cg_rows_per_block=1024, cg_gang_max=gang)
        for _ in range(2):
            system = (A, b, torch.zeros_like(b), 1e-8, 1e-8, 5, 1)
            hh.batch_run_async(x, y, off_d, off, tols, res[1], [system], cg_out, opt=opt)
            torch.cuda.synchronize()
            assert q.parse_cg_results(cg_out)[0]["status"] == q.E_DEVICE
            assert torch.equal(res[0], res[1])


def _solves(handle, stream, side, seed, iters, rounds, opt, out):
    import torch
    A = q.Csr(*workloads.poisson2d_csr(side))
    b = torch.from_numpy(workloads.normal_vector(A.n, seed)).to("cuda:0")
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(rounds):
            x = torch.zeros_like(b)
            r = handle.cg(A, b, x, 1e-300, 1e-8, iters, 1, opt, stream=stream)
            stream.synchronize()
            out.append((r["status"], r["iters"], x.cpu().numpy().tobytes()))


@pytest.mark.parametrize("sides,iters,rounds,opt",
                         [((450, 450, 500), 20, 30, None),   # no two of them fit together
                          ((1024, 450), 1500, 2, None),      # the first holds the chip for 75 ms
                          ((700, 450), 20, 15, [0, 0, 0, 0, 1])])
def test_solves_on_several_streams(sides, iters, rounds, opt):
    """Solves on streams of their own at the same time, each with its handle
    and thread, whose gangs would together need more CUs than there are: every
    one gives what it gives alone, byte for byte."""
    import threading
    import torch
    handles = [q.Qdot(0) for _ in sides]
    streams = [torch.cuda.Stream() for _ in sides]
    try:
        want = []
        for k, side in enumerate(sides):
            one = []
            _solves(handles[k], streams[k], side, k, iters, 1, opt, one)
            assert one[0][:2] == (q.E_MAXIT, iters)
            want.append(one[0])
        got = [[] for _ in sides]
        threads = [threading.Thread(target=_solves, args=(handles[k], streams[k], side, k, iters,
                                                          rounds, opt, got[k]))
                   for k, side in enumerate(sides)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        for k in range(len(sides)):
            assert len(got[k]) == rounds and all(r == want[k] for r in got[k])
    finally:
        for handle in handles:
            handle.close()


@pytest.mark.parametrize("use", [0, 1])
def test_a_system_of_one_row(h, use):
    """3 x = 6: one step from 0 gives 2 (each product and quotient rounds
    once), and the residual is 0."""
    import torch
    A = q.Csr(np.array([0, 1], np.int32), np.zeros(1, np.int32), np.full(1, 3.0))
    b = torch.full((1,), 6.0, dtype=torch.float64, device="cuda:0")
    x = torch.zeros_like(b)
    r = h.cg(A, b, x, 1e-12, 1e-10, 12, use)
    assert (r["status"], r["iters"], float(x)) == (q.OK, 1, 2.0)
    assert r["relres_true"] <= 1e-15
