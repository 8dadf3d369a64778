"""The calls whose speed matters to a user of this framework, as cases that can be timed and checked.

A case is a dict of plain values.  ``listed()`` names twelve of them, from one training step on four
qubits to a 20-qubit, 20-layer step of 500 samples; ``draw(rng)`` gives further cases of the same ranges.
``prepare`` makes what a program holds before the call (inputs on the GPU, the plan, the workspace it
keeps), ``run`` is one pass through the public entry points, ``work`` counts what a pass cannot do
without, and ``exact`` computes the same outputs in complex128 with plain torch.

Kinds of call:

  train    forward, loss in torch and adjoint backward through ``circuit_expectations`` (autograd);
           returns the expectations and the gradients of the angles and of the inputs
  infer    ``Plan.forward`` with a workspace that the program keeps
  serve    ``Plan.forward_noalloc``, the call for loops that may not allocate
  states   ``Plan.forward`` and ``Plan.backward`` from given initial states, observable (IXYZ) repeated
  mixed    ``Batch.forward`` and ``Batch.backward`` of many different circuits
"""
import math

import numpy as np
import torch

from paper_2603_02804_amd import autotune, qfuse
from paper_2603_02804_amd.workloads import CNOT, CZ, hea_gates, pauli_string

RYRZ, RXRYRZ = "RY,RZ", "RX,RY,RZ"


def listed():
    return [
        # the smallest training step: the 4-qubit, 2-layer configuration, bound by latency and launches
        case("train_4q2l", "train", 4, 2, 8, rot=RYRZ, obs=1),
        # one sample of a shallow circuit served from a loop that may not allocate
        case("serve_7q5l", "serve", 7, 5, 1, rot=RXRYRZ, obs=3),
        # a variational loop on one sample: a deep chain of small launches
        case("train_10q30l_1", "train", 10, 30, 1, rot=RXRYRZ, obs=10, loss="mean"),
        # library defaults (recompute scheme), an odd register and an odd batch
        case("train_11q37l", "train", 11, 37, 99, rot=RXRYRZ, obs=3, loss="ce", tuning="default"),
        # the 12-qubit, 100-layer, batch 1024 configuration with its tuned plan: the state fits one tile
        case("train_12q100l", "train", 12, 100, 1024, rot=RYRZ, obs=12, loss="mean"),
        # the 16-qubit, 200-layer, 4-class configuration with its tuned plan
        case("train_16q200l", "train", 16, 200, 512, rot=RXRYRZ, obs=4, loss="ce"),
        # CNOT ring, library defaults: segments are recomputed from their checkpoints
        case("train_17q25l_cnot", "train", 17, 25, 21, rot=RYRZ, obs=2, tuning="default", ring=True, ent="CNOT"),
        # the largest: the 20-qubit, 10-class configuration, its first 20 layers on half its batch (at its full
        # depth the expectations are so small that float32 holds four of their digits)
        case("train_20q20l", "train", 20, 20, 500, rot=RXRYRZ, obs=10, loss="ce"),
        # expectations only, the forward pass on its own
        case("infer_18q20l", "infer", 18, 20, 65, rot=RXRYRZ, obs=10),
        # one layer from random states on a small register and a large batch: reductions over the batch
        case("states_9q1l", "states", 9, 1, 65536, rot=RXRYRZ, ring=True),
        # the same at 20 qubits: passes and observables stream the states through memory
        case("states_20q1l", "states", 20, 1, 128, rot=RXRYRZ, ring=True),
        # many different circuits in one call (10-18 qubits, 4 samples each)
        case("mixed_64", "mixed", 18, 250, 4, rot=RYRZ, min_qubits=10, min_layers=50, circuits=64, spec=5),
    ]


def case(name, kind, qubits, layers, batch, rot=RXRYRZ, obs=1, loss="sum", tuning="tuned", ring=False, ent="CZ", **more):
    c = {"kind": kind, "qubits": qubits, "layers": layers, "batch": batch, "rot": rot, "obs": obs, "loss": loss,
         "tuning": tuning, "ring": ring, "ent": ent, **more}
    return {"name": name, **c} if name else c


# a drawn case costs at most this many amplitude-runs (the largest listed one has 2.1e11)
MOST_COST = 1.0e11


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["train", "train", "train", "infer", "serve", "states", "mixed"])
    rot = rng.choice([RYRZ, RXRYRZ])
    if kind == "mixed":
        lo = rng.randint(10, 12)
        return case("", "mixed", rng.randint(lo + 2, 17), log_int(60, 150), rng.randint(2, 4), rot=rot, min_qubits=lo,
                    min_layers=50, circuits=log_int(8, 40), spec=rng.randrange(1 << 20))
    if kind == "serve":
        n = rng.randint(4, 12)
        return case("", "serve", n, log_int(1, 40), rng.randint(1, 8), rot=rot, obs=rng.randint(1, n))
    n = rng.randint(4, 20)
    if kind == "states":
        most = max(64, min(65536, (1 << 27) >> n))
        return case("", "states", n, log_int(1, 8), log_int(8, most), rot=RXRYRZ, ring=True)
    layers = log_int(1, 150 if n <= 16 else 25)   # deeper large circuits: see the largest listed case
    most = max(1, min(1024, int(MOST_COST / (layers * n * 2.0 ** n))))
    more = {"ring": rng.random() < 0.3, "ent": rng.choice(["CZ", "CZ", "CNOT"]), "tuning": rng.choice(["tuned", "default"])}
    obs = rng.randint(1, min(n, 12))
    loss = rng.choice(["sum", "mean", "ce"]) if obs > 1 else "sum"
    return case("", kind, n, layers, log_int(1, most), rot=rot, obs=obs, loss=loss, **more)


# ---------------------------------------------------------------- circuits and inputs
def rotations(c):
    return tuple(c["rot"].split(","))


def gate_list(c, qubits, layers):
    return hea_gates(qubits, layers, rotations(c), encoding=c["kind"] != "states", ring=c["ring"],
                     entangler=CNOT if c["ent"] == "CNOT" else CZ)


def masks(c):
    """(x, z) masks of the observables: <Z_0>..<Z_{obs-1}>, or the Pauli string (IXYZ) over the register."""
    if c["kind"] == "states":
        x, z = pauli_string(("IXYZ" * (c["qubits"] // 4 + 1))[:c["qubits"]])
        return [x], [z]
    n_obs = 1 if c["kind"] == "mixed" else c["obs"]
    return [0] * n_obs, [1 << q for q in range(n_obs)]


def shapes(c):
    """(qubits, layers) of every circuit of the case."""
    if c["kind"] != "mixed":
        return [(c["qubits"], c["layers"])]
    r = np.random.default_rng(c["spec"])
    ns = r.integers(c["min_qubits"], c["qubits"] + 1, size=c["circuits"])
    ls = r.integers(c["min_layers"], c["layers"] + 1, size=c["circuits"])
    return list(zip(ns.tolist(), ls.tolist()))


def inputs(c, seed):
    """Seeded inputs on the GPU: angles ~ U[0, 2 pi), features ~ U[-pi, pi), labels, and for `states` random
    normalised initial states."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    per_layer, B = len(rotations(c)), c["batch"]
    thetas, xs = [], []
    for n, L in shapes(c):
        thetas.append(torch.rand(L * per_layer * n, generator=g, device="cuda") * (2 * math.pi))
        xs.append((torch.rand(B, n, generator=g, device="cuda") * 2 - 1) * math.pi)
    out = {"thetas": thetas, "xs": xs}
    if c["kind"] == "mixed":
        out["dEs"] = [torch.randn(B, 1, generator=g, device="cuda") for _ in thetas]
    if c["loss"] == "ce":
        out["labels"] = torch.randint(0, c["obs"], (B,), generator=g, device="cuda")
    if c["kind"] == "states":
        psi = torch.randn(B, 1 << c["qubits"], dtype=torch.complex64, generator=g, device="cuda")
        out["psi0"] = psi / torch.linalg.vector_norm(psi, dim=1, keepdim=True)
        out["dE"] = torch.randn(B, 1, generator=g, device="cuda")
    return out


def loss_of(c, E, labels):
    if c["loss"] == "ce":
        return torch.nn.functional.cross_entropy(E, labels)
    return E.mean(dim=1).sum() if c["loss"] == "mean" else E.sum()


def tuning_of(c, gates, device):
    """The tuned configuration of a known circuit, else the uncompute scheme; None: library defaults."""
    if c["tuning"] == "default":
        return None
    if c["kind"] == "states":   # a short circuit: the whole batch in one micro-batch
        return qfuse.make_tuning(uncompute=1, micro_batch=c["batch"])
    found = autotune.cached_tuning(c["qubits"], gates, len(masks(c)[0]), c["batch"], autotune.device_key(device))
    return autotune.tuning_from(found) if found else qfuse.make_tuning(uncompute=1)


def prepare(c, seed):
    dev = torch.device("cuda")
    s = {"case": c, **inputs(c, seed)}
    xm, zm = masks(c)
    circuits = []
    for (n, L), theta in zip(shapes(c), s["thetas"]):
        gates = gate_list(c, n, L)
        circuits.append(qfuse.Circuit(n, gates, theta.numel(), 0 if c["kind"] == "states" else n, zm, xm))
    if c["kind"] == "mixed":
        s["batch"] = qfuse.Batch(circuits, [c["batch"]] * len(circuits), qfuse.make_tuning(uncompute=1))
        s["ws"] = s["batch"].new_workspace(dev)
        return s
    s["theta"], s["x"] = s["thetas"][0], s["xs"][0]
    s["plan"] = qfuse.Plan(circuits[0], c["batch"], None if c["kind"] == "serve" else tuning_of(c, circuits[0].gates, dev))
    if c["kind"] in ("infer", "states"):
        s["ws"] = s["plan"].new_workspace(dev)
    if c["kind"] == "train":
        s["theta"].requires_grad_(True)
        s["x"].requires_grad_(True)
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "serve":
        return s["plan"].forward_noalloc(s["theta"], s["x"])
    if c["kind"] == "infer":
        return s["plan"].forward(s["theta"], s["x"], s["ws"])
    if c["kind"] == "states":
        E = s["plan"].forward(s["theta"], None, s["ws"], psi0=s["psi0"])
        dtheta, _ = s["plan"].backward(s["theta"], None, s["dE"], s["ws"], psi0=s["psi0"])
        return E, dtheta
    if c["kind"] == "mixed":
        E = s["batch"].forward(s["thetas"], s["xs"], s["ws"])
        dthetas, dxs = s["batch"].backward(s["thetas"], s["xs"], s["dEs"], s["ws"])
        # flat vectors, as an optimiser over all circuits takes them
        return torch.cat([e.reshape(-1) for e in E]), torch.cat(dthetas), torch.cat([d.reshape(-1) for d in dxs])
    theta, x = s["theta"], s["x"]
    theta.grad = x.grad = None
    E = qfuse.circuit_expectations(theta, x, s["plan"])
    loss_of(c, E, s.get("labels")).backward()
    return E.detach(), theta.grad, x.grad


def work(c):
    """Bytes: each input read once, each output written once.  Flops, per amplitude: one real rotation (three
    fused multiply-adds per real pair, 6 flops) per run of a qubit and one complex phase (6 flops) per layer;
    a gradient un-applies both states (twice that) and forms up to three functionals per run (4 flops each)."""
    nbytes, flops = 0.0, 0.0
    grad = c["kind"] in ("train", "states", "mixed")
    n_obs, per_layer = len(masks(c)[0]), len(rotations(c))
    for n, L in shapes(c):
        features = 0 if c["kind"] == "states" else n
        io = L * per_layer * n + c["batch"] * (features + n_obs)
        nbytes += 4.0 * io + (4.0 * (io - c["batch"] * n_obs) + 4.0 * c["batch"] * n_obs if grad else 0.0)
        if c["kind"] == "states":
            nbytes += 8.0 * c["batch"] * 2 ** n
        amps = float(c["batch"]) * 2 ** n
        flops += amps * L * (6 * n + 6)
        if grad:
            flops += amps * L * (12 * n + 12 + 4 * per_layer * n)
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------- the same outputs in complex128
# most amplitude-runs that `exact` computes: about 10 s of complex128 products on one GPU
MOST_EXACT = 2.2e11


def exact(c, seed):
    if sum(c["batch"] * L * n * 2.0 ** n for n, L in shapes(c)) > MOST_EXACT:
        return None
    s = inputs(c, seed)
    xm, zm = masks(c)
    if c["kind"] == "mixed":
        parts = []
        for (n, L), theta, x, dE in zip(shapes(c), s["thetas"], s["xs"], s["dEs"]):
            parts.append(Exact(c, n, L, theta, x, None, xm, zm).both(lambda E, dE=dE: dE.double()))
        return tuple(torch.cat([p[i].reshape(-1) for p in parts]) for i in range(3))
    X = Exact(c, c["qubits"], c["layers"], s["thetas"][0], s["xs"][0], s.get("psi0"), xm, zm)
    if c["kind"] in ("infer", "serve"):
        return X.forward()
    if c["kind"] == "states":
        return X.both(lambda E: s["dE"].double())[:2]

    def upstream(E):
        E = E.clone().requires_grad_(True)
        return torch.autograd.grad(loss_of(c, E, s.get("labels")), E)[0]

    return X.both(upstream)


class Exact:
    """Layer by layer in complex128: the rotations of a layer as Kronecker products over groups of up to five
    qubits, the entanglers as a diagonal or a permutation; gradients by the adjoint method from the groups'
    matrices sum_rest conj(lambda_i) psi_j, reduced to one qubit."""

    def __init__(self, c, n, L, theta, x, psi0, xm, zm):
        self.n, self.L, self.rots, self.B = n, L, rotations(c), c["batch"]
        self.dev = theta.device
        self.angles = theta.detach().double().reshape(L, len(self.rots), n)
        self.x, self.psi0, self.xm, self.zm = x.detach().double(), psi0, xm, zm
        count = (n + 4) // 5
        edges = [n * i // count for i in range(count + 1)]
        self.groups = [list(range(a, b)) for a, b in zip(edges, edges[1:])]
        self.index = torch.arange(1 << n, device=self.dev)
        pairs = [(q, q + 1) for q in range(n - 1)] + ([(n - 1, 0)] if c["ring"] and n > 2 else [])
        self.sign = self.gather = None
        if c["ent"] == "CNOT":
            src = self.index
            for a, b in reversed(pairs):
                src = src ^ (((src >> a) & 1) << b)
            self.gather, self.scatter = src, torch.argsort(src)
        else:
            odd = torch.zeros_like(self.index)
            for a, b in pairs:
                odd ^= (self.index >> a) & (self.index >> b) & 1
            self.sign = (1 - 2 * odd).double()
        # run matrices [L, n, 2, 2] and, for each gate of the run, dU U^dagger of its angle
        self.gates = [rotation(r, self.angles[:, j]) for j, r in enumerate(self.rots)]
        U = self.gates[0]
        for G in self.gates[1:]:
            U = G @ U
        self.kron = []
        for grp in self.groups:
            K = torch.ones(L, 1, 1, dtype=torch.complex128, device=self.dev)
            for q in reversed(grp):
                K = (K[:, :, None, :, None] * U[:, q][:, None, :, None, :]).reshape(L, K.shape[1] * 2, -1)
            self.kron.append(K)

    def entangle(self, v, back=False):
        if self.sign is not None:
            return v * self.sign
        return v[:, self.scatter if back else self.gather]

    def turn(self, v, K):
        """K on the lowest qubits of [B, 2^n], which move to the top of the index."""
        v = v.reshape(self.B, -1, K.shape[0])
        return torch.matmul(K, v.transpose(1, 2)).reshape(self.B, -1)

    def observe(self, v, k):
        """The k-th Pauli string applied to v."""
        odd = torch.zeros_like(self.index)
        src = self.index ^ self.xm[k]
        for q in range(self.n):
            if (self.zm[k] >> q) & 1:
                odd ^= (src >> q) & 1
        factor = (1j) ** bin(self.xm[k] & self.zm[k]).count("1")
        return v[:, src] * ((1 - 2 * odd).to(torch.complex128) * factor)

    def state(self):
        if self.psi0 is not None:
            v = self.psi0.to(torch.complex128)
        else:   # RY encoding of |0...0>: a product of real vectors
            v = torch.ones(self.B, 1, dtype=torch.complex128, device=self.dev)
            for q in range(self.n):
                f = torch.stack([torch.cos(self.x[:, q] / 2), torch.sin(self.x[:, q] / 2)], 1)
                v = (f[:, :, None] * v[:, None, :]).reshape(self.B, -1)
        for l in range(self.L):
            for K in self.kron:
                v = self.turn(v, K[l])
            v = self.entangle(v)
        return v

    def expect(self, v):
        return torch.stack([(v.conj() * self.observe(v, k)).sum(1).real for k in range(len(self.zm))], 1)

    def forward(self):
        return self.expect(self.state())

    def both(self, upstream):
        psi = self.state()
        E = self.expect(psi)
        g = upstream(E)
        lam = sum(2 * g[:, k:k + 1] * self.observe(psi, k) for k in range(len(self.zm)))
        grams = [torch.empty_like(K) for K in self.kron]
        kron_back = [K.conj().resolve_conj().transpose(1, 2).contiguous() for K in self.kron]
        rows = (self.B << self.n) // max(K.shape[1] for K in self.kron)
        chunks = max(k for k in range(1, min(4096, 1 + rows // 128) + 1) if rows % k == 0)
        for l in reversed(range(self.L)):
            psi, lam = self.entangle(psi, True), self.entangle(lam, True)
            for G, K in zip(grams, kron_back):
                a, b = lam.reshape(chunks, -1, K.shape[1]), psi.reshape(chunks, -1, K.shape[1])
                G[l] = torch.matmul(a.transpose(1, 2).conj().resolve_conj().contiguous(), b).sum(0)
                psi, lam = self.turn(psi, K[l]), self.turn(lam, K[l])
        M = torch.zeros(self.L, self.n, 2, 2, dtype=torch.complex128, device=self.dev)
        for grp, G in zip(self.groups, grams):
            for j, q in enumerate(grp):
                hi, lo = G.shape[1] >> (j + 1), 1 << j
                T = G.reshape(self.L, hi, 2, lo, hi, 2, lo)
                M[:, q] = torch.diagonal(torch.diagonal(T, dim1=1, dim2=4), dim1=2, dim2=4).sum((-1, -2))
        # dL/dangle = Re sum_ij M_ij (A P A^dagger)_ij (-i/2), A = the later gates of the run
        grads = []
        later = torch.eye(2, dtype=torch.complex128, device=self.dev).expand(self.L, self.n, 2, 2)
        for r, G in reversed(list(zip(self.rots, self.gates))):
            D = later @ pauli(r, self.dev) @ later.conj().transpose(-1, -2)
            grads.append((-0.5j * D * M).sum((-1, -2)).real)
            later = later @ G
        dtheta = torch.stack(grads[::-1], 1).reshape(-1)
        if self.psi0 is not None:
            return E, dtheta, None
        dx = torch.empty_like(self.x)
        for q in range(self.n):
            a, b = (v.reshape(self.B, -1, 2, 1 << q) for v in (lam, psi))
            dx[:, q] = 0.5 * (a[:, :, 1].conj() * b[:, :, 0] - a[:, :, 0].conj() * b[:, :, 1]).sum((1, 2)).real
        return E, dtheta, dx


def pauli(name, dev):
    m = {"RX": [[0, 1], [1, 0]], "RY": [[0, -1j], [1j, 0]], "RZ": [[1, 0], [0, -1]]}[name]
    return torch.tensor(m, dtype=torch.complex128, device=dev)


def rotation(name, phi):
    """cos(phi/2) I - i sin(phi/2) P, for every angle."""
    eye = torch.eye(2, dtype=torch.complex128, device=phi.device)
    return torch.cos(phi / 2)[..., None, None] * eye - 1j * torch.sin(phi / 2)[..., None, None] * pauli(name, phi.device)
