"""Layout moves in tile passes and probabilities in logical order, element by element: the smallest
states of each tile, odd sizes and layouts whose low bits go far."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def state(n, seed):
    import torch

    import paper_2608_16940_amd as P
    sv = P.StateVector(n)
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    torch.view_as_real(sv.amps).normal_(generator=gen)
    return sv


def logical_index(n, layout):
    """Logical index of every physical one."""
    import torch
    y = torch.arange(1 << n, device="cuda:0")
    x = torch.zeros_like(y)
    for q in range(n):
        x |= ((y >> int(layout[q])) & 1) << q
    return x


@pytest.mark.parametrize("n", [12, 13, 14, 17, 23, 25])
def test_layout_moves_every_amplitude(n):
    import torch
    rng = np.random.default_rng(n)
    sv = state(n, n)
    before = sv.amps.clone()
    moves = [rng.permutation(n), np.arange(n)[::-1].copy(), np.roll(np.arange(n), 1), np.arange(n)]
    for layout in moves:
        sv.permute_layout(layout)
        assert np.array_equal(sv.layout(), layout)
        assert torch.equal(sv.amps, before[logical_index(n, layout)]), (n, layout)
    sv.close()


@pytest.mark.parametrize("n", [11, 12, 13, 18, 19, 20, 24])
def test_logical_probabilities_are_exact(n):
    import torch
    rng = np.random.default_rng(100 + n)
    sv = state(n, n)
    amps = torch.view_as_real(sv.amps).double()
    want = amps[:, 0] * amps[:, 0] + amps[:, 1] * amps[:, 1]
    for layout in (np.arange(n)[::-1].copy(), rng.permutation(n), np.roll(np.arange(n), 5), np.arange(n)):
        sv.permute_layout(layout)
        assert torch.equal(sv.probs(logical=True), want)
    sv.close()
