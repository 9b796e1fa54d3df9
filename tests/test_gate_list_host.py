"""apply_gates on lists, argument marshalling only: which calls a list makes (no GPU, no library)."""
import numpy as np
import pytest

import paper_2608_16940_amd as P


class Gate:
    def __init__(self, targets, matrix=None, fail=None):
        self.targets = targets
        self.fail = fail
        self.m = np.eye(1 << len(targets), dtype=complex) if matrix is None else matrix

    @property
    def matrix(self):
        if self.fail:
            raise self.fail
        return self.m


@pytest.fixture
def sv(monkeypatch):
    calls = []

    class Lib:
        def sv_apply_gates(self, h, count, ks, targets, matrices):
            ks = np.frombuffer(ks, np.int32)
            assert len(ks) == count and len(matrices) == 16 * int((4 ** ks.astype(int)).sum())
            calls.append(("list", list(ks)))
            return 0

        def sv_apply_fused(self, h, m, t, k):
            calls.append(("apply", k))
            return 0

        def sv_free(self, h):
            return 0
    monkeypatch.setattr(P, "lib", lambda: Lib())
    s = P.StateVector.__new__(P.StateVector)
    s._h = None
    s.calls = calls
    return s


def test_what_precedes_a_gate_that_raises_is_applied(sv):
    for err in (RuntimeError("needs detach"), KeyError("theta"), TypeError("no array")):
        sv.calls.clear()
        with pytest.raises(type(err)):
            sv.apply_gates([Gate((0,)), Gate((1, 2)), Gate((3,), fail=err), Gate((4,))])
        assert sv.calls == [("apply", 1), ("apply", 2)]


def test_lists_of_wide_gates_go_one_by_one(sv):
    six = Gate(tuple(range(6)))
    sv.apply_gates([six, six, Gate((0,))])
    assert sv.calls == [("apply", 6), ("apply", 6), ("apply", 1)]
    sv.calls.clear()
    sv.apply_gates([Gate((0,)), six, Gate((1, 0)), Gate(tuple(range(5)))])
    assert sv.calls == [("list", [1, 6, 2, 5])]
    sv.calls.clear()
    sv.apply_gates([Gate((0,)), Gate(tuple(range(7)))])
    assert sv.calls == [("apply", 1), ("apply", 7)]


def test_targets_that_apply_refuses_stay_refused(sv):
    for bad in ({0}, {0: 1}, "a", b"a"):
        g = Gate((0,))
        g.targets = bad
        sv.calls.clear()
        with pytest.raises(Exception):
            sv.apply_gates([Gate((1,)), g])
        assert sv.calls == [("apply", 1)]


def test_arrays_and_lists_as_targets(sv):
    sv.apply_gates([Gate([1, 0]), Gate(np.array([2, 3])), Gate(np.array([4], np.int64)), Gate(())])
    assert sv.calls == [("list", [2, 2, 1, 0])]


def test_a_number_as_target(sv):
    g = Gate((0,))
    g.targets = 3  # what apply takes
    sv.apply_gates([g])
    assert sv.calls == [("apply", 1)]
