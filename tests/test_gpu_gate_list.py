"""apply_gates on a list against apply gate by gate: states, layouts, statistics, and errors part-way."""
import numpy as np
import pytest

from workloads import circuits as C

pytestmark = pytest.mark.gpu


def _mixed(n, count, seed):
    """Narrow gates of every kind, qubit swaps and wider gates, on any targets in any order."""
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(count):
        kind = rng.integers(0, 10)
        k = 1 if kind < 5 or n < 2 else 2
        if kind == 9 and n >= 4:
            k = int(rng.integers(3, min(n, 5) + 1))
        t = tuple(int(q) for q in rng.choice(n, k, replace=False))
        D = 1 << k
        if kind in (4, 5, 6):  # diagonal, some entries exactly 1
            d = np.exp(1j * rng.uniform(0, 6, D))
            d[rng.random(D) < 0.5] = 1.0
            m = np.diag(d)
        elif kind == 7 and k == 2:
            m = C.swap()
        else:
            m = np.linalg.qr(rng.standard_normal((D, D)) + 1j * rng.standard_normal((D, D)))[0]
        out.append(C.Gate("g", t, m))
    return out


@pytest.mark.parametrize("n", [1, 3, 4, 5, 9, 10, 11, 12, 13, 16, 21, 22, 23])
@pytest.mark.parametrize("narrow", [False, True])
def test_list_equals_gates_one_by_one(n, narrow):
    import torch
    from paper_2608_16940_amd import StateVector
    gates = C.brickwork(n, 12, 3) if narrow and n > 1 else _mixed(n, 150, n)
    a, b = StateVector(n), StateVector(n)
    g = torch.Generator(device="cuda:0").manual_seed(n)
    torch.view_as_real(a.amps).normal_(0.0, 2.0 ** (-(n + 1) / 2), generator=g)
    b.amps.copy_(a.amps)
    a.apply_gates(gates)
    for x in gates:
        b.apply(x.matrix, x.targets)
    assert list(a.layout()) == list(b.layout())
    sa, sb = a.stats(), b.stats()
    sa.pop("launches"), sb.pop("launches")
    assert sa == sb
    # a sweep rounds each amplitude within four units of 2^-24 per term and the two orders differ by commuting gates only
    d = (a.amps - b.amps).to(torch.complex128).norm() / b.amps.to(torch.complex128).norm()
    assert float(d) <= 8 * 2.0 ** -24 * sum(1 << len(x.targets) for x in gates)


def test_what_precedes_a_bad_gate_is_applied():
    from paper_2608_16940_amd import StateVector, SvError
    n = 12
    gates = C.brickwork(n, 2, 5)
    bad = C.Gate("bad", (n,), gates[0].matrix)
    a, b = StateVector(n), StateVector(n)
    a.reset(), b.reset()
    with pytest.raises(SvError):
        a.apply_gates(gates + [bad] + gates)
    b.apply_gates(gates)
    a.sync(), b.sync()
    assert (a.copy_out() == b.copy_out()).all()
    assert a.stats()["gate_sweeps"] == b.stats()["gate_sweeps"]


@pytest.mark.parametrize("n", [3, 4, 12, 20])
def test_unfused_plan_equals_the_list(n):
    import torch
    from paper_2608_16940_amd import Plan, StateVector
    gates = C.brickwork(n, 10, 7)
    plan = Plan.greedy(n, gates, 1)
    a, b = StateVector(n), StateVector(n)
    g = torch.Generator(device="cuda:0").manual_seed(n)
    torch.view_as_real(a.amps).normal_(0.0, 2.0 ** (-(n + 1) / 2), generator=g)
    b.amps.copy_(a.amps)
    plan.run(a)
    for x in plan.blocks():
        b.apply(x["matrix"], x["targets"])
    sa, sb = a.stats(), b.stats()
    sa.pop("launches"), sb.pop("launches")
    assert sa == sb
    d = (a.amps - b.amps).to(torch.complex128).norm() / b.amps.to(torch.complex128).norm()
    assert float(d) <= 8 * 2.0 ** -24 * sum(1 << len(x.targets) for x in gates)


def test_long_and_odd_lists():
    from paper_2608_16940_amd import StateVector
    n = 12
    gates = C.brickwork(n, 100, 9)  # more than one call's gates
    seven = np.linalg.qr(np.random.default_rng(1).standard_normal((128, 128)))[0].astype(complex)
    gates = gates[:700] + [C.Gate("wide", tuple(range(7)), seven)] + gates[700:]
    a, b = StateVector(n), StateVector(n)
    a.reset(), b.reset()
    a.apply_gates([])
    a.apply_gates(gates)
    b.apply_gates(iter(gates))  # not a list: one by one
    assert a.stats()["by_variant"] == b.stats()["by_variant"]
    x, y = a.copy_out(), b.copy_out()
    assert np.linalg.norm(x - y) <= 8 * 2.0 ** -24 * sum(1 << len(g.targets) for g in gates)
