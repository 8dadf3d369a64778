"""The small launches that end a circuit's sequence in a mixed batch are shared by all
circuits of a group at its last steps, and every circuit still gets its own results."""
import numpy as np
import pytest

import plancheck
from paper_2603_02804_amd.workloads import mixed, z_observables


@pytest.mark.parametrize("n, layers, tuning", [
    (1, (5, 5), {}),                                        # one circuit: its own sequence
    (6, (1, 12), dict(fusion_depth=1)),                     # every circuit ends at another step
    (5, (2, 9), dict(uncompute=1, ckpt_interval=2, fusion_depth=1)),  # assemblies between the passes too
])
def test_trailing_small_launches_are_shared(n, layers, tuning):
    ws = mixed(n, (13, 13), layers, 2, 31)
    xm, zm = z_observables([0])
    dEs = [np.random.default_rng(7).normal(size=(2, 1)).astype(np.float32) for _ in ws]
    circuits = [(c.n_qubits, c.gates, len(c.theta), c.n_qubits, zm) for c in ws]
    Es, dth, dxs, st = plancheck.batch_run(circuits, [2] * n, [c.theta for c in ws], [c.x for c in ws], dEs, **tuning)
    single = {"epoch_fill": 2, "fusion_depth": 12, **tuning}
    passes = []
    for i, c in enumerate(ws):
        passes.append(plancheck.stats(c.n_qubits, c.gates, len(c.theta), c.n_qubits, zm, 2, **single)["passes"])
        E1, dth1, dx1 = plancheck.run(c.n_qubits, c.gates, c.theta, c.x, zm, dEs[i], **single)
        np.testing.assert_array_equal(Es[i], E1)
        np.testing.assert_array_equal(dth[i], dth1)
        np.testing.assert_array_equal(dxs[i], dx1)
    # one tile shape in at most two groups; a group's forward is coefficients, phase
    # events, the passes of its longest circuit and one shared expectation reduction
    assert st["fwd_launches"] <= min(n, 2) * (max(passes) + 3)
