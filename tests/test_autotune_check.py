"""The autotuner compares the call that it times, not only the route that
returns the classes (CPU: a handle whose two routes disagree)."""
import pytest

torch = pytest.importorskip("torch")

from paper_2105_00115_amd import autotune  # noqa: E402

RESULT = {"count": [1, 2, 3, 4], "n_zero": 0, "e_min": -3, "e_max": 5, "t": -20, "flags": 0,
          "n_bins": 9, "bound_rel": 1e-7, "status": 0, "value": 1.5}


class Handle:
    """Both routes give RESULT, but for what `wrong` changes in the timed one
    (by options: None or the guaranteed mode's)."""

    def __init__(self, wrong=None, guarded=False):
        self.wrong, self.guarded = wrong or {}, guarded

    def set_tune(self, *a, **k):
        pass

    def qdot_classes(self, x, y, tol):
        return torch.zeros(10, dtype=torch.uint8), torch.arange(5), dict(RESULT)

    def qdot(self, x, y, tol, opt=None):
        r = dict(RESULT)
        if (opt is not None) == self.guarded:
            r.update(self.wrong)
        return r


CFG = (2, 1, 2, 1, 8, 1, 0, 8, 256)


def _check(handle):
    x = torch.ones(10, dtype=torch.float64)
    ref = autotune._reference(Handle(), x, x, 1e-6)
    autotune._check_same(handle, x, x, 1e-6, CFG, ref)


def test_agreeing_routes_pass():
    _check(Handle())
    _check(Handle({"value": 1.5 + 1e-14}))  # sum |x y| = 10: its rounding


@pytest.mark.parametrize("guarded", [False, True])
@pytest.mark.parametrize("wrong", [{"count": [1, 2, 4, 3]}, {"t": -21}, {"flags": 1},
                                   {"bound_rel": 2e-7}, {"value": 1.5 + 1e-12}])
def test_a_wrong_timed_route_is_found(wrong, guarded):
    with pytest.raises(autotune.ShapeChanged):
        _check(Handle(wrong, guarded))
