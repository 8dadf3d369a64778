"""qf_forward_noalloc for plans whose workspace ends close to the library's array: the epoch
tables in their own place, over the parts of the workspace that only a backward uses, or in
memory of the plan; every result equals qf_forward's bit for bit, and a refusal names the
size that was compared."""
import ctypes

import numpy as np
import pytest

import plancheck as pc
from paper_2603_02804_amd.workloads import draw_inputs, hea_gates

LIMIT = 64 << 20
CASES = {   # qubits, layers, samples, tuning
    "own place": (12, 200, 8, dict(micro_batch=1, uncompute=1, ckpt_interval=2)),
    "functionals": (12, 200, 271, dict(micro_batch=24, uncompute=1, ckpt_interval=2)),
    "functionals, tables of few rows": (13, 40, 142, dict(uncompute=1)),
    "adjoint states": (12, 200, 273, dict(micro_batch=24, uncompute=1, ckpt_interval=2)),
    "plan": (12, 200, 285, dict(micro_batch=1, uncompute=1, ckpt_interval=2)),
    "refused": (12, 200, 300, dict(micro_batch=1, uncompute=1, ckpt_interval=2)),
}


def layout(name):
    """(workspace, start of the tables, their bytes, where the forward alone keeps them)"""
    n, L, B, tun = CASES[name]
    gates = hea_gates(n, L, ("RX", "RY", "RZ"))
    d, keep = pc._desc(n, gates, L * 3 * n, n, [1])
    t, out = pc.make_tuning(**tun), (ctypes.c_int64 * 20)()
    assert pc.lib().qfc_stats(ctypes.byref(d), B, ctypes.byref(t), out, 20) == 0
    return out[11], out[17], out[18], out[19]


@pytest.mark.parametrize("name", CASES)
def test_place_cpu(name):
    ws, start, size, at = layout(name)
    if name == "own place":
        assert at == start and ws <= LIMIT
    elif name == "plan":
        assert at == -1 and start <= LIMIT
    elif name == "refused":
        assert at == -1 and start > LIMIT
    else:   # where the tables would reach beyond the array, they lie inside it, over other parts
        assert start + size > LIMIT >= at + size and 0 < at < start


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_noalloc_gpu(name):
    import torch
    from paper_2603_02804_amd import qfuse
    dev = torch.device("cuda:0")
    n, L, B, tun = CASES[name]
    theta, x, _ = draw_inputs(n, L * 3 * n, B, n)
    circ = qfuse.Circuit(n, hea_gates(n, L, ("RX", "RY", "RZ")), len(theta), n, [1])
    plan = qfuse.Plan(circ, B, qfuse.make_tuning(**tun))
    ws = plan.new_workspace(dev)
    th, xx = torch.tensor(theta, device=dev), torch.tensor(x, device=dev)
    E = plan.forward(th, xx, ws)
    if name == "refused":
        with pytest.raises(qfuse.QFuseError) as e:
            plan.forward_noalloc(th, xx)
        assert e.value.status == 3 and str(layout(name)[1]) in str(e.value)
        return
    for _ in range(2):
        assert torch.equal(plan.forward_noalloc(th, xx), E)
