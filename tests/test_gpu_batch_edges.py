"""Batched circuits at the edges of the packs and of the passes, against the oracle."""
import numpy as np
import pytest

import oracle
from workloads import circuits as C

pytestmark = pytest.mark.gpu


def _ladder(n, depth, seed, cnots=True):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(depth):
        out += [C.Gate("ry", (q,), C.ry(rng.uniform(0, 6))) for q in range(n)]
        if cnots:
            out += [C.Gate("cnot", (q, q + 1), C.cnot()) for q in range(n - 1)]
    return out


# states in LDS: one circuit to sixteen per workgroup, CNOT runs of no, two and many gates; states in
# passes: no gate, one pass, several
@pytest.mark.parametrize("sizes", [[1] * 3, [2, 3, 4] * 6, [9] * 17, [10] * 16 + [11], [12] * 5, [13] * 3, [14] * 2,
                                   [15, 14, 3], [16, 15], [18, 17]])
def test_batch_edges(sizes):
    from paper_2608_16940_amd.batch import Batch
    circs = []
    for i, n in enumerate(sizes):
        depth = (1 if n > 16 else 3) + i % 2
        gates = _ladder(n, depth, i, cnots=i % 3 != 2)
        if n > 14 and len(circs) == 0:
            gates += _ladder(n, 1, 99)[::-1]
        circs.append((n, gates))
        if n > 14:
            circs.append((n, []))  # stays |0...0>
            circs.append((n, [C.Gate("h", (1,), C.ry(0.3)), C.Gate("cnot", (1, 2), C.cnot())]))
    b = Batch(circs).allocate()
    for z in (b.run(), b.prepare().launch(), b.launch()):
        for i, (n, gates) in enumerate(circs):
            ref = oracle.run(n, gates)
            got = b.state(i)
            # every gate rounds an amplitude within four units of 2^-24
            tol = 8 * 2.0 ** -24 * max(1, len(gates))
            assert np.abs(got - ref).max() <= tol
            assert abs(z[i] - oracle.expect_z(ref, 0)) <= 2 * tol
