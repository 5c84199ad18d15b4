"""The paper's speedup and efficiency need the parameter selection and the
computation phase timed apart."""
import pytest

import paper_2105_00115_amd as q
import workloads
from paper_2105_00115_amd import studies

pytestmark = pytest.mark.gpu


def _times(h, n):
    import torch
    x, y = workloads.paper_dist_torch(n, 9, 3, "B")
    out = torch.zeros(q.RESULT_BYTES, dtype=torch.uint8, device="cuda:0")
    h.qdot_async(x, y, 1e-6, out)
    torch.cuda.synchronize()
    h.timing_read()
    h.timing_enable(True)
    for _ in range(5):
        h.qdot_async(x, y, 1e-6, out)
    torch.cuda.synchronize()
    h.timing_enable(False)
    t = h.timing_read()
    return {k: t[k] / t["qdot_calls"] for k in ("scan_ms", "cut_ms", "acc_ms", "fin_ms")}


@pytest.mark.parametrize("n", [1000, 100_000, 1_000_000, 10_000_000, (1 << 24) + 4])
def test_selection_and_computation_have_kernels_of_their_own(n):
    """Selection and combine take a launch each: 2 us or more past the gap of
    two events with nothing between them, which is what the default shapes
    show there (the shortest launch on this card takes about 4 us)."""
    with q.Qdot(0) as default, studies.separate_kernels(q.Qdot(0)) as h:
        gap, t = _times(default, n), _times(h, n)
        assert t["cut_ms"] > gap["cut_ms"] + 0.002, (gap, t)
        assert t["fin_ms"] > 0.0 and t["acc_ms"] > gap["fin_ms"] + 0.002, (gap, t)
        # the scan reads both vectors whole (at most 8 TB/s)
        assert t["scan_ms"] >= 16.0 * n / 8e12 * 1e3


def test_effectiveness_study_uses_them(monkeypatch, tmp_path):
    seen = []

    def record(h, *a, **k):
        seen.append([h.get_tune(b)[-1] for b in range(4)])
        return {}

    monkeypatch.setattr(studies, "study_e2", record)
    assert studies.main(["--study", "e2", "--scale", "small", "--out",
                         str(tmp_path / "s.json")]) == 0
    assert seen == [[512] * 4]
