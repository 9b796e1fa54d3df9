"""A plan on a density handle against its blocks one by one: the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# handles below and above the size from which gates share passes; blocks of every width a chain takes
@pytest.mark.parametrize("n,k", [(5, 6), (8, 4), (9, 4), (9, 6), (10, 5), (10, 6), (11, 6), (12, 4), (12, 7)])
def test_plan_equals_blocks_bit_for_bit(n, k):
    import torch
    import paper_2608_16940_amd as P
    rng = np.random.default_rng(n * 10 + k)
    gates = []
    for i in range(14):
        w = min(int(rng.integers(3, k + 1)), 2 * n)
        t = rng.choice(2 * n, w, replace=False) if i % 3 else rng.integers(0, 2 * n - w + 1) + rng.permutation(w)
        D = 1 << w
        m = np.linalg.qr(rng.standard_normal((D, D)) + 1j * rng.standard_normal((D, D)))[0]
        if i == 7:
            m = np.diag(np.exp(1j * rng.uniform(0, 6, D)))
        gates.append(P.SuperGate("g", tuple(int(q) for q in t), m, i == 7))
    plan = P.Plan.greedy(2 * n, gates, k)
    a, b = P.DensityMatrix(n), P.DensityMatrix(n)
    g = torch.Generator(device="cuda:0").manual_seed(n)
    torch.view_as_real(a.amps).normal_(0.0, 2.0 ** (-n), generator=g)
    b.amps.copy_(a.amps)
    for _ in range(2):
        plan.run(a)
        for x in plan.blocks():
            P.StateVector.apply(b, x["matrix"], x["targets"])
    assert torch.equal(a.amps, b.amps)
    assert list(a.layout()) == list(b.layout())
    sa, sb = a.stats(), b.stats()
    sa.pop("launches"), sb.pop("launches")
    assert sa == sb
