"""Fused tile passes (several blocks of a plan in one pass over the state) against the oracle.

Every tile size the builder picks (one tile of 2^10..2^14 amplitudes, 2^12 tiles of cache-sized
states, 2^14 tiles above), five- and six-bit gates on any targets, narrower ones, diagonals on tile
and outside bits, more gates than operands stay resident, and diagonals alone.
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2608_16940_amd as P
    P.lib()
    return P


def diagonal(n, k, rng):
    t = tuple(int(q) for q in rng.choice(n, k, replace=False))
    return W.Gate("diag", t, np.diag(np.exp(1j * rng.uniform(0, 2 * np.pi, 1 << k))), diag=True)


def sequence(n, rng, kind):
    if kind == "diag":
        return [diagonal(n, int(rng.integers(4, 9)), rng) for _ in range(12)]
    gates = []
    for i in range(24):
        if rng.random() < 0.4:
            gates.append(diagonal(n, int(rng.integers(1, 6)), rng))
        elif kind == "near":  # neighbours, as fused circuits have: many gates to a tile
            k = int(rng.integers(1, 7))
            s = int(rng.integers(0, n - k + 1))
            gates.append(W.random_dense(n, k, rng, tuple(range(s, s + k))))
        else:
            gates.append(W.random_dense(n, int(rng.integers(1, 7)), rng))
    return gates


@pytest.mark.parametrize("kind", ["near", "any", "diag"])
@pytest.mark.parametrize("n", [10, 11, 12, 13, 14, 15, 17, 21, 22])
def test_passes_match_oracle(P, n, kind):
    rng = np.random.default_rng([n, ord(kind[0])])
    prep = [W.Gate("su2", (q,), W.haar_su2(rng)) for q in range(n)]
    gates = sequence(n, rng, kind)
    plan = P.Plan.greedy(n, gates, 1)  # wider than the cap: every gate a block of its own
    sv = P.StateVector(n)
    sv.apply_gates(prep)
    plan.run(sv)
    st = sv.stats()
    assert st["launches"] - len(prep) < len(gates)  # some blocks shared a pass
    got = oracle.decode(sv.physical_state(), sv.layout())
    m = oracle.metrics(oracle.run(n, prep + gates), got)
    print("n", n, kind, m, flush=True)
    # one FP32 rounding of each amplitude and of each gate entry or table entry per gate, doubled
    assert m["rel_l2"] <= (len(prep) + len(gates)) * 2 ** -22
    sv.close()
