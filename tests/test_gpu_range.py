"""Upstream gradients and initial states near the ends of the float range on the GPU against
the oracle: half turns (their unscaled rotations would grow a state by up to 2^25 each),
random angles and per-sample half turns.  Everything is linear in dE and in |psi0|^2, so the
oracle runs on the unscaled values."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.oracle import Oracle  # noqa: E402
from paper_2603_02804_amd import qfuse  # noqa: E402
from paper_2603_02804_amd.workloads import CNOT, CZ, hea_gates, z_observables  # noqa: E402

pytestmark = pytest.mark.gpu
PI = np.pi


def angles(rng, kind, shape):
    some = rng.choice([PI, -PI, 3 * PI, PI - 1e-5, 1.0], shape)
    return {"half_turns": np.full(shape, PI), "some": some, "random": rng.uniform(0, 2 * PI, shape)}[kind].astype(np.float32)


@pytest.mark.parametrize("kind", ["half_turns", "some", "random"])
@pytest.mark.parametrize("scale_dE,scale_psi", [(2.0 ** 116, None), (2.0 ** -100, None), (1.0, 2.0 ** 44),
                                                (2.0 ** 60, 2.0 ** 28), (2.0 ** 20, 2.0 ** -40)])
@pytest.mark.parametrize("n,tun,general", [
    (4, {}, False), (9, {}, True), (12, {}, False), (14, dict(uncompute=1), False), (13, dict(ckpt_interval=2), True),
    (6, dict(reg_qubits=1), False), (8, dict(reg_qubits=3), False), (12, dict(reg_qubits=5), False),
])
def test_range(n, tun, general, scale_dE, scale_psi, kind):
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n)
    L, B, rots = 3, 3, ("RX", "RY", "RZ")
    gates = hea_gates(n, L, rots, ring=True, entangler=CNOT if n % 2 else CZ)
    P = L * len(rots) * n
    theta, x = angles(rng, kind, P), angles(rng, kind, (B, n))
    xm, zm = z_observables([0, n - 1])
    if general:
        xm = np.array([1, 2], np.uint64)
    dE = rng.normal(size=(B, 2)).astype(np.float32)
    psi0 = None
    if scale_psi:
        psi0 = rng.normal(size=(B, 1 << n)) + 1j * rng.normal(size=(B, 1 << n))
        psi0 = (psi0 / np.linalg.norm(psi0, axis=1, keepdims=True)).astype(np.complex64)
    plan = qfuse.Plan(qfuse.Circuit(n, gates, P, n, zm, xm), B, qfuse.make_tuning(**tun))
    ws = plan.new_workspace(dev)
    th, xx = torch.tensor(theta, device=dev), torch.tensor(x, device=dev)
    p0 = torch.tensor(psi0, device=dev) * scale_psi if scale_psi else None
    E = plan.forward(th, xx, ws, psi0=p0)
    dth, dx = plan.backward(th, xx, torch.tensor(dE, device=dev) * scale_dE, ws, psi0=p0)
    Eo, dtho, dxo = Oracle().backward(n, gates, theta, x, xm, zm, dE, psi0=psi0)
    e = (scale_psi or 1.0) ** 2
    # each run turns the state with an error of a few 2^-24 (angle, scale, rounding), the
    # adjoint carries two such states; observables and the functionals are at most quadratic
    tol, lam = plan.info.n_runs * 4 * 2.0 ** -23, 2 * np.abs(dE).sum()
    assert np.abs(E.cpu().double().numpy() / e - Eo).max() <= tol
    assert np.abs(dth.cpu().double().numpy() / (e * scale_dE) - dtho).max() <= tol * lam
    assert np.abs(dx.cpu().double().numpy() / (e * scale_dE) - dxo).max() <= tol * lam


def test_range_batch():
    """The same in a mixed batch, whose circuits take their own routes."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(5)
    ns, L, B, scale = (10, 12, 13), 3, 2, 2.0 ** 116
    zm = z_observables([0])[1]
    cs = [(n, hea_gates(n, L, ("RY", "RZ")), angles(rng, k, L * 2 * n), angles(rng, k, (B, n)))
          for n, k in zip(ns, ("half_turns", "random", "some"))]
    dEs = [rng.normal(size=(B, 1)).astype(np.float32) for _ in ns]
    batch = qfuse.Batch([qfuse.Circuit(n, g, len(t), n, zm) for n, g, t, _ in cs], [B] * 3, qfuse.make_tuning(uncompute=1))
    ws = batch.new_workspace(dev)
    th, xx = [torch.tensor(c[2], device=dev) for c in cs], [torch.tensor(c[3], device=dev) for c in cs]
    batch.forward(th, xx, ws)
    dth, dx = batch.backward(th, xx, [torch.tensor(d, device=dev) * scale for d in dEs], ws)
    for (n, g, t, x), d, a, b in zip(cs, dEs, dth, dx):
        _, dtho, dxo = Oracle().backward(n, g, t, x, np.zeros(1, np.uint64), zm, d)
        tol = (L + 1) * n * 4 * 2.0 ** -23 * 2 * np.abs(d).sum()
        assert np.abs(a.cpu().double().numpy() / scale - dtho).max() <= tol
        assert np.abs(b.cpu().double().numpy() / scale - dxo).max() <= tol
