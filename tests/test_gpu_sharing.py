"""That gates share launches where they should, and that the kernels they bypass are still covered.

A call on a list or a plan is held against the same gates one by one on a second handle: fewer
launches, the same state.  Statistics by lowering are predicted on the host for shared passes, so
only the launch count shows whether a pass ran.
"""
import numpy as np
import pytest
import torch  # noqa: F401  the library shares its HIP runtime: loaded first

import oracle
import workloads as W
from workloads import circuits as C

pytestmark = pytest.mark.gpu


def launched(sv, call):
    before = sv.stats()["launches"]
    call()
    return sv.stats()["launches"] - before


def handles(make, seed):
    """Two handles in the same random state of norm one."""
    a, b = make(), make()
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    torch.view_as_real(a.amps).normal_(0.0, (2.0 * a.amps.numel()) ** -0.5, generator=g)
    b.amps.copy_(a.amps)
    return a, b


def one_by_one(sv, gates):
    from paper_2608_16940_amd import StateVector
    for x in gates:
        StateVector.apply(sv, x.matrix, x.targets)


def distance(a, b):
    x, y = a.amps.to(torch.complex128), b.amps.to(torch.complex128)
    return float((x - y).norm() / y.norm())


def diagonal(n, k, rng, entries=None):
    t = tuple(int(q) for q in rng.choice(n, k, replace=False))
    d = np.exp(1j * rng.uniform(0, 6, 1 << k)) if entries is None else rng.choice(entries, 1 << k)
    return C.Gate("d", t, np.diag(d), diag=True)


def sequence(n, kind, rng):
    if kind == "diagonal":
        return [diagonal(n, int(rng.integers(4, 9)), rng) for _ in range(12)]
    out = []
    for _ in range(24):
        k = int(rng.integers(1, 7))
        if rng.random() < 0.4:
            out.append(diagonal(n, min(k, 5), rng))
        elif kind == "near":
            s = int(rng.integers(0, n - k + 1))
            out.append(W.random_dense(n, k, rng, tuple(range(s, s + k))))
        else:
            out.append(W.random_dense(n, k, rng))
    return out


# every tile size; FP32 bounds: one rounding of each amplitude and of each gate or table entry, both sides
@pytest.mark.parametrize("kind", ["near", "any", "diagonal"])
@pytest.mark.parametrize("n", [10, 11, 12, 14, 17, 21, 22])
def test_blocks_of_a_plan_share_passes(n, kind):
    from paper_2608_16940_amd import Plan, StateVector
    rng = np.random.default_rng([n, len(kind)])
    gates = sequence(n, kind, rng)
    a, b = handles(lambda: StateVector(n), n)
    plan = Plan.greedy(n, gates, 1)
    fused, single = launched(a, lambda: plan.run(a)), launched(b, lambda: one_by_one(b, gates))
    print(n, kind, "launches", fused, "of", single, flush=True)
    assert fused < min(single, len(gates))
    assert list(a.layout()) == list(b.layout())
    assert distance(a, b) <= 2 * len(gates) * 2.0 ** -22


@pytest.mark.parametrize("n", [4, 10, 12, 16, 22])
def test_narrow_gates_of_a_list_share_passes(n):
    from paper_2608_16940_amd import StateVector
    gates = C.brickwork(n, 6, n)
    a, b = handles(lambda: StateVector(n), n)
    fused, single = launched(a, lambda: a.apply_gates(gates)), launched(b, lambda: one_by_one(b, gates))
    assert fused <= single // 8
    assert distance(a, b) <= 8 * 2.0 ** -24 * sum(1 << len(x.targets) for x in gates)


# From 25 qubits on few controlled phases are swept alone: on qubits above a cache line's each visits a
# quarter of the state
@pytest.mark.parametrize("n,count,launches", [(24, 2, 1), (25, 2, 2), (25, 3, 3), (25, 4, 1)])
def test_few_phases_on_a_large_state(n, count, launches):
    from paper_2608_16940_amd import StateVector
    gates = [C.Gate("cp", (8 + i, n - 1 - i), C.cphase(0.3 + i), True) for i in range(count)]
    a, b = handles(lambda: StateVector(n), n)
    assert launched(a, lambda: a.apply_gates(gates)) == launches
    one_by_one(b, gates)
    assert distance(a, b) <= 8 * 2.0 ** -24 * 4 * count
    a.close(), b.close()


@pytest.mark.parametrize("n", [9, 10, 12])
def test_density_blocks_share_passes(n):
    from paper_2608_16940_amd import DensityMatrix, Plan, SuperGate
    rng = np.random.default_rng(n)
    gates = []
    for _ in range(10):
        t = rng.integers(0, 2 * n - 4) + rng.permutation(4)
        m = np.linalg.qr(rng.standard_normal((16, 16)) + 1j * rng.standard_normal((16, 16)))[0]
        gates.append(SuperGate("g", tuple(int(q) for q in t), m))
    plan = Plan.greedy(2 * n, gates, 1)
    blocks = [C.Gate("b", x["targets"], x["matrix"]) for x in plan.blocks()]  # targets in the plan's order
    a, b = handles(lambda: DensityMatrix(n), n)
    assert launched(a, lambda: plan.run(a)) < launched(b, lambda: one_by_one(b, blocks)) == len(gates)
    assert torch.equal(a.amps, b.amps)


UNITS = np.array([1, -1, 1j, -1j])


@pytest.mark.parametrize("n", [10, 12, 13, 16, 21, 22])
def test_exact_diagonals_share_passes_in_bf16x3(n):
    """Entries 1, -1, i, -i: nothing is rounded, so a pass gives the bits of the sweeps."""
    from paper_2608_16940_amd import Plan, StateVector
    rng = np.random.default_rng(n)
    gates = [diagonal(n, int(rng.integers(3, 7)), rng, UNITS) for _ in range(14)]
    plan = Plan.greedy(n, gates, 1)
    a, b = handles(lambda: StateVector(n), n)
    a.set_precision("bf16x3"), b.set_precision("bf16x3")
    assert launched(a, lambda: plan.run(a)) < launched(b, lambda: one_by_one(b, gates))
    assert torch.equal(a.amps, b.amps)


@pytest.mark.parametrize("n", [12, 15, 21, 22])
def test_exact_diagonals_between_dense_gates_in_bf16x3(n):
    from paper_2608_16940_amd import Plan, StateVector
    rng = np.random.default_rng(n)
    prep = [C.Gate("su2", (q,), C.haar_su2(rng)) for q in range(n)]
    gates = []
    for _ in range(6):
        gates.append(W.random_dense(n, int(rng.integers(5, 7)), rng))
        gates += [diagonal(n, int(rng.integers(3, 6)), rng, UNITS) for _ in range(3)]
    plan = Plan.greedy(n, gates, 1)
    sv, one = StateVector(n), StateVector(n)
    for s in (sv, one):
        s.set_precision("bf16x3")
        s.apply_gates(prep)
    assert launched(sv, lambda: plan.run(sv)) < launched(one, lambda: one_by_one(one, gates))
    m = oracle.metrics(oracle.run(n, prep + gates), oracle.decode(sv.physical_state(), sv.layout()))
    print(n, m, flush=True)
    assert m["rel_l2"] <= 1e-4  # the arithmetic's bound for 168 sweeps


@pytest.mark.parametrize("n", [1, 2, 4, 9, 12, 17])
def test_diagonals_one_by_one_take_the_streaming_kernel(n):
    """Lists of narrow diagonals run as programs; gate by gate the kernel itself is what is checked."""
    import paper_2608_16940_amd as P
    rng = np.random.default_rng(60 + n)
    prep = [C.Gate("su2", (q,), C.haar_su2(rng)) for q in range(n)]
    gates = [diagonal(n, k, rng) for k in range(1, min(n, 8) + 1)] + [diagonal(n, 1, rng) for _ in range(2)]
    sv = P.StateVector(n)
    sv.apply_gates(prep)
    before = sv.stats()
    one_by_one(sv, gates)
    after = sv.stats()
    d = P._native.VARIANT["diag"]
    assert after["by_variant"][d] - before["by_variant"][d] == len(gates)
    assert after["launches"] - before["launches"] >= len(gates)
    m = oracle.metrics(oracle.run(n, prep + gates), oracle.decode(sv.physical_state(), sv.layout()))
    assert m["rel_l2"] <= (len(prep) + len(gates)) * 2.0 ** -22
