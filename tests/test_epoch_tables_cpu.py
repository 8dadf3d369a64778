"""The CPU execution of the planner's programs takes what the pass kernels take: run groups
and diagonal items from the epoch tables and records, functionals from chunked column sums.
Enough samples for several chunks, shared and per-sample runs in one group, half turns on
states whose unscaled rotations would leave the float range, against the oracle."""
import numpy as np
import pytest

import plancheck as pc
from oracle.oracle import Oracle
from paper_2603_02804_amd.workloads import CNOT, CZ, RX, RY, RZ, z_observables


@pytest.mark.parametrize("n,B,ent,turns,tun", [
    (5, 300, CZ, False, {}),                                     # one tile, several chunks of rows
    (8, 40, CNOT, False, dict(tile_qubits=5, ckpt_interval=2)),  # eight tiles, segments
    (7, 130, CZ, False, dict(micro_batch=100, tile_qubits=5)),   # a last micro-batch of fewer rows
    (6, 3, CZ, True, {}),
    (9, 2, CNOT, True, dict(tile_qubits=7, uncompute=1)),
    (7, 2, CZ, True, dict(reg_qubits=5)),
    (5, 2, CNOT, True, dict(reg_qubits=2, tile_qubits=4)),
])
def test_against_oracle(n, B, ent, turns, tun):
    rng = np.random.default_rng(10 * n + B)
    rows, k = [], 0
    for layer in range(3):
        for q in range(n):
            if (q + layer) % 2:   # per-sample runs beside shared ones
                rows.append((RY, q, -1, -1, q))
            for kind in ((RX, RY, RZ), (RY, RZ), (RZ, RY))[(q + layer) % 3]:
                rows.append((kind, q, -1, k, -1))
                k += 1
        rows += [(ent, q, (q + 1) % n, -1, -1) for q in range(n)]
    gates = np.asarray(rows, np.int32)
    pick = np.float32([np.pi, -np.pi, np.pi - 1e-5, 0.0, 1.0])
    theta = (rng.choice(pick, k) if turns else rng.uniform(0, 2 * np.pi, k)).astype(np.float32)
    x = (rng.choice(pick, (B, n)) if turns else rng.uniform(-np.pi, np.pi, (B, n))).astype(np.float32)
    psi0 = rng.normal(size=(B, 1 << n)) + 1j * rng.normal(size=(B, 1 << n))
    psi0 = (psi0 / np.linalg.norm(psi0, axis=1, keepdims=True)).astype(np.complex64)
    s = 2.0 ** 44 if turns else 1.0
    xm, zm = z_observables([0, n - 1])
    dE = rng.normal(size=(B, 2)).astype(np.float32)
    E, dth, dx = pc.run(n, gates, theta, x, zm, dE, psi0=psi0 * np.float32(s), **tun)
    Eo, dtho, dxo = Oracle().backward(n, gates, theta, x, xm, zm, dE, psi0=psi0)
    # a few 2^-24 per run for the state and the adjoint, whose norm bounds the rest
    tol = pc.stats(n, gates, k, n, zm, B, **tun)["runs"] * 4 * 2.0 ** -23
    assert np.abs(E / s ** 2 - Eo).max() <= tol
    assert np.abs(dth / s ** 2 - dtho).max() <= tol * 2 * np.abs(dE).sum()
    assert np.abs(dx / s ** 2 - dxo).max() <= tol * 2 * np.abs(dE).sum()
