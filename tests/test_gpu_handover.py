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
