"""Gradients where the RY part of a run is exactly the identity, or exactly a half turn: RY
angles of zero beside RZ angles (zero-initialised parameters, zero features), RY pairs that
cancel, in runs of RY gates followed by RZ gates, whose adjoint forms no X functional.  On
the CPU execution of the planner's programs and on the GPU, against the oracle."""
import numpy as np
import pytest

from oracle.oracle import Oracle
from paper_2603_02804_amd.workloads import CNOT, CZ, RX, RY, RZ, z_observables

PATTERNS = {"ry_rz": [(RY, RZ)], "ryry_rzrz": [(RY, RY, RZ, RZ)], "mixed": [(RY, RZ), (RX,), (RZ, RY), (RY, RY, RZ)]}
CASES = [(n, tun, pattern, zeros, ent)
         for n, tun in [(1, {}), (4, {}), (9, {}), (13, dict(uncompute=1)), (12, dict(reg_qubits=5)), (8, dict(reg_qubits=3))]
         for pattern in PATTERNS for zeros in ("all", "some", "pairs", "half_turns") for ent in (CZ, CNOT)]


def circuit(n, pattern, zeros, ent, L=3, B=3):
    rng = np.random.default_rng(100 * n + len(pattern) + len(zeros))
    rows, theta = [], []
    x = rng.choice(np.float32([0, 0.7]), (B, n)).astype(np.float32)
    x[0] = 0
    for layer in range(L):
        for q in range(n):
            if layer != 1:   # (the middle layer's runs are shared by all samples)
                rows.append((RY, q, -1, -1, q))
            before = len(theta)
            for kind in PATTERNS[pattern][(q + layer) % len(PATTERNS[pattern])]:
                rows.append((kind, q, -1, len(theta), -1))
                angle = rng.uniform(-np.pi, np.pi)
                if kind == RY:
                    prev = theta[-1] if len(theta) > before else 0.0
                    angle = {"all": 0.0, "some": rng.choice([0.0, angle]), "pairs": -prev if prev else rng.choice([0.0, -0.7, angle]),
                             "half_turns": np.pi}[zeros]
                theta.append(np.float32(angle))
        rows += [(ent, q, q + 1, -1, -1) for q in range(n - 1)]
    xm, zm = z_observables([0, n - 1])
    dE = rng.normal(size=(B, 2)).astype(np.float32)
    return np.asarray(rows, np.int32), np.asarray(theta, np.float32), x, xm, zm, dE


def check(got, n, gates, theta, x, xm, zm, dE, runs):
    _, dtho, dxo = Oracle().backward(n, gates, theta, x, xm, zm, dE)
    # a few 2^-24 per run for the state and the adjoint, times the adjoint's norm
    tol = runs * 4 * 2.0 ** -23 * 2 * np.abs(dE).sum()
    assert np.abs(got[0] - dtho).max() <= tol
    assert np.abs(got[1] - dxo).max() <= tol


@pytest.mark.parametrize("n,tun,pattern,zeros,ent", CASES)
def test_zero_angles_cpu(n, tun, pattern, zeros, ent):
    import plancheck as pc
    c = gates, theta, x, xm, zm, dE = circuit(n, pattern, zeros, ent)
    _, dth, dx = pc.run(n, gates, theta, x, zm, dE, **tun)
    check((dth, dx), n, *c, pc.stats(n, gates, len(theta), n, zm, len(x), **tun)["runs"])


@pytest.mark.gpu
@pytest.mark.parametrize("n,tun,pattern,zeros,ent", CASES)
def test_zero_angles_gpu(n, tun, pattern, zeros, ent):
    import torch
    from paper_2603_02804_amd import qfuse
    c = gates, theta, x, xm, zm, dE = circuit(n, pattern, zeros, ent)
    dev = torch.device("cuda:0")
    plan = qfuse.Plan(qfuse.Circuit(n, gates, len(theta), n, zm), len(x), qfuse.make_tuning(**tun))
    ws = plan.new_workspace(dev)
    th, xx = torch.tensor(theta, device=dev), torch.tensor(x, device=dev)
    plan.forward(th, xx, ws)
    dth, dx = plan.backward(th, xx, torch.tensor(dE, device=dev), ws)
    check((dth.cpu().numpy(), dx.cpu().numpy()), n, *c, plan.info.n_runs)
