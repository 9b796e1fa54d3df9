"""Bound plans of every route against plan.run: the same bits, also replayed as a graph."""
import numpy as np
import pytest
import torch  # noqa: F401  the library shares its HIP runtime: loaded first

from workloads import circuits as C

pytestmark = pytest.mark.gpu


def _narrow(n, seed):
    """One-qubit gates and diagonals on one or two qubits: the plan runs as programs."""
    rng = np.random.default_rng(seed)
    out = []
    for i in range(90):
        if i % 3 == 0:
            t = tuple(int(q) for q in rng.choice(n, 2, replace=False))
            out.append(C.Gate("d", t, np.diag(np.exp(1j * rng.uniform(0, 6, 4))), diag=True))
        else:
            out.append(C.Gate("u", (int(rng.integers(0, n)),), C.haar_su2(rng)))
    return out


def _replays(plan, a, b, reset, same_launches=True):
    """plan.run on a; bound on b: once eagerly, then three graph replays with eager work between them."""
    reset(a)
    plan.run(a)
    want = a.physical_state()
    reset(b)
    bound = plan.bind(b)
    bound.run()
    np.testing.assert_array_equal(b.physical_state(), want)
    assert list(a.layout()) == list(b.layout())
    for rep in range(3):
        reset(b)
        bound.run_graph()
        np.testing.assert_array_equal(b.physical_state(), want, err_msg="replay %d" % rep)
        b.norm()
    sa, sb = a.stats(), b.stats()
    if not same_launches:
        sa.pop("launches"), sb.pop("launches")
    assert sa == sb
    bound.close()


@pytest.mark.parametrize("n", [4, 11, 12, 15, 22])
def test_unfused_plan(n):
    from paper_2608_16940_amd import Plan, StateVector
    plan = Plan.greedy(n, _narrow(n, n), 1)
    _replays(plan, StateVector(n), StateVector(n), lambda sv: sv.reset())


def test_unfused_plan_needs_no_operand_memory():
    import ctypes
    from paper_2608_16940_amd import Plan, StateVector, lib
    sv = StateVector(14)
    need = ctypes.c_size_t(1)
    assert lib().sv_bound_bytes(sv._h, Plan.greedy(14, _narrow(14, 1), 1)._h, ctypes.byref(need)) == 0
    assert need.value == 0


@pytest.mark.parametrize("n,k", [(8, 4), (9, 6), (11, 5)])
def test_density_plan(n, k):
    from paper_2608_16940_amd import DensityMatrix, Plan, SuperGate
    rng = np.random.default_rng(n)
    gates = []
    for i in range(12):
        w = int(rng.integers(4, k + 1))
        t = rng.integers(0, 2 * n - w + 1) + rng.permutation(w)
        m = np.linalg.qr(rng.standard_normal((1 << w, 1 << w)) + 1j * rng.standard_normal((1 << w, 1 << w)))[0]
        gates.append(SuperGate("g", tuple(int(q) for q in t), m))
    plan = Plan.greedy(2 * n, gates, k)

    def reset(dm):
        dm.reset()
        for q in range(2 * n):  # every amplitude at work
            dm.apply(C.ry(0.3 + 0.1 * q), (q,))
    _replays(plan, DensityMatrix(n), DensityMatrix(n), reset, same_launches=False)
