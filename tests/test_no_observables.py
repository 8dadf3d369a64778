"""Circuits without observables: plans and mixed batches are accepted, the forward writes
nothing and every gradient is zero, in all modes, with one and with several partial sums
per sample and tile."""
import numpy as np
import pytest

from paper_2603_02804_amd.workloads import draw_inputs, hea_gates

B = 3


def circuit(n):
    gates = hea_gates(n, 2, ("RY", "RZ"))
    theta, x, _ = draw_inputs(n, 4 * n, B, n)
    return gates, theta, x


def test_batch_cpu():
    import plancheck as pc
    cs = [(n, *circuit(n)) for n in (10, 12, 14)]
    none = [np.zeros((B, 0), np.float32)] * 3
    _, dth, dx, _ = pc.batch_run([(n, g, len(t), n, []) for n, g, t, _ in cs], [B] * 3, [c[2] for c in cs],
                                 [c[3] for c in cs], none)
    assert all(not d.any() for d in dth + dx)


@pytest.mark.gpu
@pytest.mark.parametrize("n,tun", [(9, {}), (12, {}), (15, {}), (12, dict(mode=1)), (12, dict(mode=2))])
def test_plan_gpu(n, tun):
    import torch
    from paper_2603_02804_amd import qfuse
    dev = torch.device("cuda:0")
    gates, theta, x = circuit(n)
    plan = qfuse.Plan(qfuse.Circuit(n, gates, len(theta), n, []), B, qfuse.make_tuning(**tun))
    ws = plan.new_workspace(dev)
    th, xx = torch.tensor(theta, device=dev, dtype=plan.dtype), torch.tensor(x, device=dev, dtype=plan.dtype)
    E = torch.full((4,), 7.0, device=dev, dtype=plan.dtype)   # (nothing is read from or written to it)
    plan.forward(th, xx, ws, E=E)
    dth, dx = plan.backward(th, xx, E, ws)
    assert not dth.any() and not dx.any() and bool((E == 7).all())


@pytest.mark.gpu
def test_batch_gpu():
    import torch
    from paper_2603_02804_amd import qfuse
    dev = torch.device("cuda:0")
    cs = [(n, *circuit(n)) for n in (10, 12, 14)]
    batch = qfuse.Batch([qfuse.Circuit(n, g, len(t), n, []) for n, g, t, _ in cs], [B] * 3)
    ws = batch.new_workspace(dev)
    th, xx = [torch.tensor(c[2], device=dev) for c in cs], [torch.tensor(c[3], device=dev) for c in cs]
    E, s = [torch.full((4,), 7.0, device=dev) for _ in cs], torch.cuda.current_stream().cuda_stream
    qfuse.qf_batch_forward(batch.handle, th, xx, E, ws, ws.numel(), s)
    dth, dx = batch.backward(th, xx, E, ws)
    assert all(not d.any() for d in dth + dx) and all(bool((e == 7).all()) for e in E)
