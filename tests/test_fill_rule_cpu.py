"""The default end-of-pass threshold on circuits that the entanglers serialise: the
planner keeps the cheapest of its schedules, and that schedule's programs (run by the
CPU execution of its programs) agree with the oracle."""
import numpy as np
import pytest

import plancheck as pc
from oracle.oracle import Oracle
from paper_2603_02804_amd.workloads import CNOT, CZ, draw_inputs, hea_gates, z_observables

E_TOL, G_TOL = 1e-4, 1e-3


@pytest.mark.parametrize("n,L,ent,ring,tun", [
    (13, 3, CNOT, True, {}),                                      # one non-local qubit
    (15, 2, CNOT, True, dict(tile_qubits=10, ckpt_interval=2)),
    (14, 3, CNOT, False, dict(uncompute=1)),
    (9, 3, CNOT, True, dict(tile_qubits=6, reg_qubits=2)),        # R < 4
    (14, 3, CZ, True, {}),                                        # the threshold R stays
])
def test_default_threshold(n, L, ent, ring, tun):
    gates = hea_gates(n, L, ("RY", "RZ"), ring=ring, entangler=ent)
    theta, x, _ = draw_inputs(40 + n, L * 2 * n, 2, n)
    xm, zm = z_observables([0, n - 1])
    dE = np.random.default_rng(n).normal(size=(2, 2))
    E, dth, dx = pc.run(n, gates, theta, x, zm, dE, **tun)
    Eo, dtho, dxo = Oracle().backward(n, gates, theta, x, xm, zm, dE)
    assert np.abs(E - Eo).max() <= E_TOL
    assert np.abs(dth - dtho).max() <= G_TOL * np.abs(dtho).max()
    assert np.abs(dx - dxo).max() <= G_TOL * np.abs(dxo).max()
    passes = [pc.stats(n, gates, len(theta), n, zm, 2, epoch_fill=f, **tun)["passes"] for f in (0, -1, 4)]
    if ent == CNOT and ring and "reg_qubits" not in tun:   # (two runs are a full epoch for R = 2)
        assert passes[0] <= passes[1] + 4 and passes[0] < passes[2]
    if ent == CZ:
        assert passes[0] == passes[2]
