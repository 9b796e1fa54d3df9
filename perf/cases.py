"""The calls this framework is timed on: what a program that simulates circuits with it makes.

Each case is one call (or the few calls that belong together) through the
package's public entry points, from the smallest states, where launches and
host work count, to the 8 GiB state of the headline circuit:

* gates      a circuit handed over gate by gate (``StateVector.apply_gates``);
* graph      a plan bound to one small state and replayed as a HIP graph;
* plan       a fused plan run on a state (``Plan.greedy`` / ``Plan.learned``,
             FP32 or BF16x3), optionally from |0...0> and ending in a QFT;
* density    a noisy circuit on a density matrix, channels fused by a plan;
* batch      many small circuits in one launch;
* measure    probabilities in logical order, the norm and samples of a state;
* layout     moving a state to other qubit layouts;
* train      one training step of the planner's cost model.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_16940_amd as P
import workloads as W
from paper_2608_16940_amd import costmodel
from paper_2608_16940_amd.batch import Batch
from workloads import noise

DEV = "cuda:0"
KRAUS_P = 1e-3


def listed():
    return [
        # a program that steps through a 12-qubit circuit: every launch and host call counts
        {"name": "gates_n12", "kind": "gates", "n": 12, "depth": 8},
        # the 20-qubit circuit applied gate by gate (the repository's C1 workload)
        {"name": "gates_n20", "kind": "gates", "n": 20, "depth": 20},
        # a small circuit evaluated over and over by replaying its bound plan (a variational loop)
        {"name": "graph_n16", "kind": "graph", "n": 16, "depth": 12, "k": 5},
        # an ordinary run on a cache-sized state with an odd number of qubits
        {"name": "plan_n23", "kind": "plan", "n": 23, "depth": 12, "k": 5, "planner": "greedy", "prec": "fp32",
         "qft": False},
        # the headline circuit: N=30, 24 brickwork layers and the QFT, greedy fusion to 5 qubits
        {"name": "headline_n30", "kind": "plan", "n": 30, "depth": 24, "k": 5, "planner": "greedy", "prec": "fp32",
         "qft": True},
        # the same family under the learned planner, whose blocks are six qubits wide
        {"name": "learned_n28", "kind": "plan", "n": 28, "depth": 16, "k": 7, "planner": "learned", "prec": "fp32",
         "qft": False},
        # wide blocks in the BF16x3 arithmetic that a caller can choose
        {"name": "bf16x3_n28", "kind": "plan", "n": 28, "depth": 16, "k": 7, "planner": "greedy", "prec": "bf16x3",
         "qft": False},
        # a 13-qubit density matrix under a noisy circuit
        {"name": "density_n13", "kind": "density", "n": 13, "depth": 4, "k": 6},
        # a parameter sweep over small circuits of mixed sizes
        {"name": "batch_512", "kind": "batch", "count": 512, "n_lo": 10, "n_hi": 18, "d_lo": 4, "d_hi": 12},
        # reading a state out after a QFT, whose closing swaps leave the layout reversed
        {"name": "measure_n28", "kind": "measure", "n": 28, "shots": 10000},
        # moving a large state between two arbitrary layouts
        {"name": "layout_n29", "kind": "layout", "n": 29},
        # one step of fitting the cost model to the sweep timings of a machine
        {"name": "train_1712", "kind": "train", "rows": 1712},
    ]


def draw(rng):
    kind = rng.choice(["gates", "graph", "plan", "plan", "plan", "density", "batch", "measure", "layout", "train"])
    if kind == "gates":
        return {"kind": kind, "n": rng.randint(8, 21), "depth": rng.randint(2, 20)}
    if kind == "graph":
        return {"kind": kind, "n": rng.randint(10, 22), "depth": rng.randint(2, 16), "k": rng.randint(3, 6)}
    if kind == "plan":
        prec = rng.choice(["fp32", "fp32", "bf16x3"])
        planner = rng.choice(["greedy", "greedy", "learned"])
        return {"kind": kind, "n": rng.randint(14, 29), "depth": rng.randint(2, 16),
                "k": 7 if planner == "learned" else rng.randint(3, 7), "planner": planner, "prec": prec,
                "qft": rng.random() < 0.4}
    if kind == "density":
        return {"kind": kind, "n": rng.randint(5, 14), "depth": rng.randint(1, 6), "k": rng.randint(4, 6)}
    if kind == "batch":
        lo = rng.randint(6, 16)
        return {"kind": kind, "count": int(round(16 * 32 ** rng.random())), "n_lo": lo,
                "n_hi": rng.randint(lo, 18), "d_lo": rng.randint(2, 6), "d_hi": rng.randint(6, 16)}
    if kind == "measure":
        return {"kind": kind, "n": rng.randint(10, 28), "shots": int(10 ** rng.uniform(1, 5))}
    if kind == "layout":
        return {"kind": kind, "n": rng.randint(12, 29)}
    return {"kind": kind, "rows": int(round(100 * 40 ** rng.random()))}


# ---------------------------------------------------------------- inputs
def _random_state(n, seed, out=None):
    """A normalised Gaussian state: every amplitude of the size a deep circuit leaves."""
    amps = torch.empty(1 << n, dtype=torch.complex64, device=DEV) if out is None else out
    gen = torch.Generator(device=DEV).manual_seed(seed)
    torch.view_as_real(amps).normal_(0.0, 2.0 ** (-(n + 1) / 2), generator=gen)
    return amps


def _circuit(case, seed):
    gates = W.brickwork(case["n"], case["depth"], seed)
    if case.get("qft"):
        gates += W.qft(case["n"])
    return gates


def _circuits(case, seed):
    """Parameter-ladder circuits as (n, depth, theta[depth, n], phi[depth, n]): the shapes belong to
    the case, the angles to the seed."""
    shape = np.random.default_rng([case["count"], case["n_lo"], case["n_hi"], case["d_lo"], case["d_hi"]])
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(case["count"]):
        n = int(shape.integers(case["n_lo"], case["n_hi"] + 1))
        d = int(shape.integers(case["d_lo"], case["d_hi"] + 1))
        out.append((n, d, rng.uniform(0, 2 * math.pi, (d, n)), rng.uniform(0, 2 * math.pi, (d, n))))
    return out


def _layouts(case, seed):
    rng = np.random.default_rng(seed)
    return rng.permutation(case["n"]), rng.permutation(case["n"])


def _training_rows(case, seed):
    """Rows shaped like the cost model's: scaled features in [0, 1] and log times of a few units."""
    rng = np.random.default_rng(seed)
    X = rng.uniform(0, 1, (case["rows"], costmodel.NIN)).astype(np.float32)
    y = (1.0 + X @ rng.standard_normal(costmodel.NIN) * 0.5 + 0.1 * rng.standard_normal(case["rows"]))
    return X, y.astype(np.float32)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("gates", "plan"):
        sv = P.StateVector(case["n"], DEV)
        gates = _circuit(case, seed)
        if not case.get("qft"):
            _random_state(case["n"], seed, sv.amps)
        if kind == "gates":
            return {"kind": kind, "sv": sv, "gates": gates}
        sv.set_precision(case["prec"])
        if case["planner"] == "learned":
            plan = P.Plan.learned(case["n"], gates, costmodel.load()[0])
        else:
            plan = P.Plan.greedy(case["n"], gates, case["k"])
        return {"kind": kind, "sv": sv, "plan": plan, "from_zero": case["qft"]}
    if kind == "graph":
        sv = P.StateVector(case["n"], DEV)
        bound = P.Plan.greedy(case["n"], _circuit(case, seed), case["k"]).bind(sv)
        return {"kind": kind, "sv": sv, "bound": bound}
    if kind == "density":
        dm = P.DensityMatrix(case["n"], DEV)
        chans = noise.noisy_brickwork(case["n"], case["depth"], KRAUS_P, seed)
        plan = P.Plan.greedy(2 * case["n"], P.superop_gates(case["n"], chans), case["k"])
        return {"kind": kind, "dm": dm, "plan": plan}
    if kind == "batch":
        circs = []
        for n, d, th, ph in _circuits(case, seed):
            gates = []
            for layer in range(d):
                for q in range(n):
                    gates.append(W.Gate("ry", (q,), W.circuits.ry(th[layer, q])))
                    gates.append(W.Gate("rz", (q,), W.circuits.rz(ph[layer, q]), True))
                gates += [W.Gate("cnot", (q, q + 1), _CNOT) for q in range(n - 1)]
            circs.append((n, gates))
        return {"kind": kind, "batch": Batch(circs).allocate(DEV).prepare()}
    if kind == "measure":
        sv = P.StateVector(case["n"], DEV)
        for q in range(case["n"] // 2):
            sv.apply(W.circuits.swap(), (q, case["n"] - 1 - q))
        _random_state(case["n"], seed, sv.amps)
        return {"kind": kind, "sv": sv, "seed": seed, "shots": case["shots"]}
    if kind == "layout":
        sv = P.StateVector(case["n"], DEV)
        _random_state(case["n"], seed, sv.amps)
        return {"kind": kind, "sv": sv, "layouts": _layouts(case, seed)}
    X, y = _training_rows(case, seed)
    net = costmodel.DeviceMLP(costmodel.init_params(seed), case["rows"], DEV)
    return {"kind": kind, "net": net, "X": torch.from_numpy(X).to(DEV), "y": torch.from_numpy(y).to(DEV)}


_CNOT = W.circuits.cnot()


def run(state):
    kind = state["kind"]
    if kind == "gates":
        state["sv"].apply_gates(state["gates"])
        return state["sv"].amps
    if kind == "plan":
        if state["from_zero"]:
            state["sv"].reset()
        state["plan"].run(state["sv"])
        return state["sv"].amps
    if kind == "graph":
        state["sv"].reset()
        state["bound"].run_graph()
        return state["sv"].amps
    if kind == "density":
        dm = state["dm"]
        dm.reset()
        state["plan"].run(dm)
        return {"rho": dm.amps, "probs": dm.probs()}
    if kind == "batch":
        z0 = state["batch"].launch()
        return {"z0": z0, "states": state["batch"].states}
    if kind == "measure":
        sv = state["sv"]
        return {"probs": sv.probs(), "norm": sv.norm(), "shots": sv.sample(state["seed"], state["shots"])}
    if kind == "layout":
        for layout in state["layouts"]:
            state["sv"].permute_layout(layout)
        return state["sv"].amps
    net = state["net"]
    net.forward(state["X"])
    net.backward(state["X"], state["y"])
    net.adam(lr=3e-3)
    return {"y": net.y, "loss": net.loss, "grads": net.g, "params": net.p}


# ---------------------------------------------------------------- the work of one pass
def _gate_flops(gates, dim):
    """Arithmetic of the gates one by one: 14 flops per amplitude for a 2x2 factor, one complex
    product on the quarter of the state that a controlled phase changes."""
    dense = sum(1 for g in gates if g.kind in ("su2", "h"))
    phases = sum(1 for g in gates if g.kind == "cp")
    return dim * (14.0 * dense + 1.5 * phases)


def work(case):
    kind = case["kind"]
    if kind in ("gates", "plan", "graph"):
        dim = float(1 << case["n"])
        from_zero = kind == "graph" or case.get("qft")
        return {"bytes": (8.0 if from_zero else 16.0) * dim, "flops": _gate_flops(_circuit(case, 0), dim)}
    if kind == "density":
        n, dim = case["n"], float(1 << (2 * case["n"]))
        chans = noise.noisy_brickwork(n, case["depth"], KRAUS_P, 0)
        # a unitary acts on rows and on columns; two-qubit depolarising mixes a 4x4 block (16 entries)
        flops = sum(28.0 * dim if c.kind == "su2" else (8.0 * dim if c.kind == "depolarizing" else 0.0) for c in chans)
        return {"bytes": 8.0 * dim + 8.0 * (1 << n), "flops": flops}
    if kind == "batch":
        circs = _circuits(case, 0)
        return {"bytes": sum(8.0 * (1 << n) + 8.0 for n, _, _, _ in circs),
                "flops": sum(14.0 * n * d * (1 << n) for n, d, _, _ in circs)}
    if kind == "measure":
        dim = float(1 << case["n"])
        return {"bytes": 16.0 * dim + 8.0 * case["shots"], "flops": 3.0 * dim}
    if kind == "layout":
        return {"bytes": 2 * 16.0 * (1 << case["n"]), "flops": 0.0}
    nin, hid, rows = costmodel.NIN, costmodel.HID, case["rows"]
    params = nin * hid + hid + hid * hid + hid + hid + 1
    return {"bytes": 4.0 * (rows * (nin + 2) + 6 * params), "flops": 6.0 * rows * params}


# ---------------------------------------------------------------- the same in 64 bits
def _apply64(psi, gate):
    """A one-qubit gate, or a diagonal two-qubit phase, in place on a complex128 state."""
    m = np.asarray(gate.matrix)
    if len(gate.targets) == 1:
        v = psi.view(-1, 2, 1 << gate.targets[0])
        a = v[:, 0] * complex(m[0, 0])
        a.add_(v[:, 1], alpha=complex(m[0, 1]))
        b = v[:, 0] * complex(m[1, 0])
        b.add_(v[:, 1], alpha=complex(m[1, 1]))
        v[:, 0] = a
        v[:, 1] = b
        return
    lo, hi = sorted(gate.targets)
    v = psi.view(-1, 2, 1 << (hi - lo - 1), 2, 1 << lo)
    v[:, 1, :, 1].mul_(complex(m[3, 3]))


def _exact_circuit(case, seed):
    if case.get("qft"):
        return None  # a fused block may carry the QFT's swaps: the stored order is the planner's
    gates = _circuit(case, seed)
    if len(gates) * (1 << case["n"]) > 3e11:
        return None
    if case["kind"] == "graph":
        psi = torch.zeros(1 << case["n"], dtype=torch.complex128, device=DEV)
        psi[0] = 1.0
    else:
        psi = _random_state(case["n"], seed).to(torch.complex128)
    for g in gates:
        _apply64(psi, g)
    return psi


def _exact_density(case, seed):
    n = case["n"]
    if n > 13:
        return None
    rho = torch.zeros(1 << (2 * n), dtype=torch.complex128, device=DEV)
    rho[0] = 1.0
    for c in noise.noisy_brickwork(n, case["depth"], KRAUS_P, seed):
        if c.kind == "su2":
            q, u = c.targets[0], c.kraus[0]
            _apply64(rho, W.Gate("u", (q,), u))
            _apply64(rho, W.Gate("u", (q + n,), u.conj()))
        elif c.kind == "cz":
            a, b = c.targets
            _apply64(rho, W.Gate("cz", (a, b), W.circuits.cz()))
            _apply64(rho, W.Gate("cz", (a + n, b + n), W.circuits.cz()))
        else:
            # rho -> (1 - 16 p / 15) rho + 4 p / 15 Tr_ab(rho) (x) 1, on neighbours a < b = a + 1
            a = min(c.targets)
            v = rho.view(1 << (n - a - 2), 4, 1 << (n - 2), 4, 1 << a)
            tr = v[:, 0, :, 0] + v[:, 1, :, 1] + v[:, 2, :, 2] + v[:, 3, :, 3]
            rho.mul_(1.0 - 16.0 * KRAUS_P / 15.0)
            for i in range(4):
                v[:, i, :, i].add_(tr, alpha=4.0 * KRAUS_P / 15.0)
    probs = rho.view(1 << n, 1 << n).diagonal().real.clamp_min(0.0)
    return {"rho": rho, "probs": probs}


def _exact_batch(case, seed):
    circs = _circuits(case, seed)
    offs = np.cumsum([0] + [1 << n for n, _, _, _ in circs])
    states = torch.empty(int(offs[-1]), dtype=torch.complex128, device=DEV)
    z0 = np.zeros(len(circs))
    for n in sorted({c[0] for c in circs}):
        idx = [i for i, c in enumerate(circs) if c[0] == n]
        # after the CNOTs (0,1), (1,2), ... bit q of the new index is the parity of the old bits 0..q
        x = torch.arange(1 << n, device=DEV)
        src = x ^ ((x << 1) & ((1 << n) - 1))
        for part in range(0, len(idx), 64):
            ids = idx[part:part + 64]
            psi = torch.zeros(len(ids), 1 << n, dtype=torch.complex128, device=DEV)
            psi[:, 0] = 1.0
            for layer in range(max(circs[i][1] for i in ids)):
                live = [j for j, i in enumerate(ids) if layer < circs[i][1]]
                sub = psi[live]
                for q in range(n):
                    th = torch.tensor([circs[ids[j]][2][layer, q] for j in live], device=DEV, dtype=torch.float64)
                    ph = torch.tensor([circs[ids[j]][3][layer, q] for j in live], device=DEV, dtype=torch.float64)
                    c, s = torch.cos(th / 2), torch.sin(th / 2)
                    e = torch.polar(torch.ones_like(ph), -ph / 2)
                    v = sub.view(len(live), -1, 2, 1 << q)
                    sh = (len(live), 1, 1)
                    a = (e * c).view(sh) * v[:, :, 0] - (e * s).view(sh) * v[:, :, 1]
                    b = (e.conj() * s).view(sh) * v[:, :, 0] + (e.conj() * c).view(sh) * v[:, :, 1]
                    v[:, :, 0] = a
                    v[:, :, 1] = b
                psi[live] = sub[:, src]
            for j, i in enumerate(ids):
                states[int(offs[i]):int(offs[i + 1])] = psi[j]
                p = psi[j].abs().square().view(-1, 2).sum(0)
                z0[i] = float(p[0] - p[1])
    return {"z0": z0, "states": states}


def _reindex(n, source_bit):
    """Index tensor whose entry y has bit b equal to bit source_bit[b] of y."""
    y = torch.arange(1 << n, device=DEV)
    x = torch.zeros_like(y)
    for b, p in enumerate(source_bit):
        x |= ((y >> int(p)) & 1) << b
    return x


def _exact_train(case, seed):
    X, y = _training_rows(case, seed)
    W1, b1, W2, b2, W3, b3 = costmodel.split_params(costmodel.init_params(seed).astype(np.float64))
    X, y = X.astype(np.float64), y.astype(np.float64)
    z1 = X @ W1 + b1
    h1 = np.maximum(z1, 0)
    z2 = h1 @ W2 + b2
    h2 = np.maximum(z2, 0)
    out = (h2 @ W3 + b3)[:, 0]
    dy = (out - y) / len(y)
    d2 = dy[:, None] * W3[:, 0] * (z2 > 0)
    d1 = (d2 @ W2.T) * (z1 > 0)
    g = np.concatenate([(X.T @ d1).ravel(), d1.sum(0), (h1.T @ d2).ravel(), d2.sum(0), h2.T @ dy, [dy.sum()]])
    loss = np.array([0.5 * np.mean((out - y) ** 2)])
    # the first Adam step moves a parameter by the sign of its gradient, so where that is rounding alone
    # (a dead unit) the step has no value of its own
    return {"y": out, "loss": loss, "grads": g, "params": None}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("gates", "plan", "graph"):
        return _exact_circuit(case, seed)
    if kind == "density":
        return _exact_density(case, seed)
    if kind == "batch":
        return _exact_batch(case, seed)
    if kind == "measure":
        n = case["n"]
        amps = _random_state(n, seed)
        p = torch.view_as_real(amps).double().square().sum(-1)
        norm = float(p.sum())
        return {"probs": p[_reindex(n, range(n - 1, -1, -1))], "norm": norm, "shots": None}
    if kind == "layout":
        last = _layouts(case, seed)[1]
        return _random_state(case["n"], seed)[_reindex(case["n"], last)].to(torch.complex128)
    return _exact_train(case, seed)
