"""Performance cases of the simulator: the calls its users make, over the
range of sizes and options they make them with.

A case is a dict of plain values; `kind` selects what one pass does:

  gate     one sv_apply_gate / sv_apply_controlled_gate on a state
  circuit  a state reset to |0...0> and one circuit through sv_apply_circuit
  step     the same followed by the norm and a 2^20-amplitude read-back
  batch    many independent small circuits through sv_batch_run
  pauli    the terms of a transverse-field Ising Hamiltonian on a lattice
  reads    the norm, a marginal distribution and samples of a state
  train    epochs of training the fusion cost model

Each kind has at least one listed case; `draw` gives further ones.  `exact`
recomputes the outputs in float64 / complex128 with plain torch.
"""
import ctypes
import math

import numpy as np
import torch

import circuits as C
from paper_2602_09604_amd import sv

READ_BACK = 1 << 20  # amplitudes a step reads back


def listed():
    return [
        # one gate of an interactive session or a variational loop on a small
        # state: nothing but the latency of the call
        {"name": "gate_1q_12", "kind": "gate", "n": 12, "k": 1, "controls": 0, "low": False},
        # a wide dense gate on a state far larger than the caches
        {"name": "gate_5q_28", "kind": "gate", "n": 28, "k": 5, "controls": 0, "low": False},
        # a circuit at the default options on a state held in the caches (the
        # 4x5 depth-14 grid of the tests and the benchmark)
        {"name": "grid20_default", "kind": "circuit", "family": "grid", "rows": 4, "cols": 5, "depth": 14,
         "fusion": "greedy", "max_k": 4, "precision": "fp32_valu", "graph": False},
        # the same circuit as a serving loop runs it: fused wide, split FP16,
        # the kept graph relaunched
        {"name": "grid20_graph", "kind": "circuit", "family": "grid", "rows": 4, "cols": 5, "depth": 14,
         "fusion": "block", "max_k": 6, "precision": "fp16x3", "graph": True},
        # a circuit at the default options on a state streamed from memory
        {"name": "grid28_default", "kind": "circuit", "family": "grid", "rows": 4, "cols": 7, "depth": 20,
         "fusion": "greedy", "max_k": 4, "precision": "fp32_valu", "graph": False},
        # the benchmark's step on the 30-qubit 5x6 depth-20 grid: learned
        # fusion, split FP16, norm and read-back
        {"name": "grid30_step", "kind": "step", "family": "grid", "rows": 5, "cols": 6, "depth": 20,
         "fusion": "learned", "max_k": 6, "precision": "fp16x3", "graph": False},
        # every gate as its own pass: the plain FP32 reference run
        {"name": "grid26_unfused", "kind": "circuit", "family": "grid", "rows": 2, "cols": 13, "depth": 6,
         "fusion": "none", "max_k": 1, "precision": "fp32_valu", "graph": False},
        # a QFT in phase fusion (runs of controlled phases as one sweep each)
        {"name": "qft28_phase", "kind": "circuit", "family": "qft", "rows": 1, "cols": 28, "depth": 1,
         "fusion": "phase", "max_k": 5, "precision": "fp16x3", "graph": False},
        # a parameter sweep: many RY-RZ-CNOT ansatz circuits of mixed sizes
        {"name": "batch48", "kind": "batch", "count": 48, "n_min": 10, "n_max": 22, "layers": 8, "max_k": 4,
         "fusion": "block"},
        # the energy of a variational state: every term of a lattice
        # Hamiltonian (ZZ on the couplers, X on the qubits)
        {"name": "ising20", "kind": "pauli", "rows": 4, "cols": 5},
        # reading a finished state: norm, 10-qubit marginal, 100000 shots
        {"name": "reads28", "kind": "reads", "n": 28, "measured": 10, "shots": 100000},
        # training the fusion cost model on the benchmark's augmented corpus
        {"name": "train7200", "kind": "train", "samples": 7200, "epochs": 20},
    ]


def draw(rng):
    kind = rng.choice(("gate", "gate", "circuit", "circuit", "circuit", "batch", "pauli", "reads", "train"))
    if kind == "gate":
        n = rng.randint(8, 28)
        return {"kind": kind, "n": n, "k": rng.randint(1, 6), "controls": rng.choice((0, 0, 1, 2)),
                "low": rng.random() < 0.4}
    if kind == "circuit":
        family = rng.choice(("grid", "grid", "qv", "qft"))
        fusion = rng.choice(("greedy", "greedy", "greedy", "block", "learned", "phase", "none"))
        if family == "grid":
            rows, cols = rng.choice(((2, 5), (3, 4), (2, 7), (3, 5), (4, 4), (3, 6), (4, 5), (3, 7), (2, 11), (4, 6),
                                     (5, 5), (2, 13), (3, 9)))
        else:
            rows, cols = 1, rng.randint(10, 26 if family == "qft" else 25)
        return {"kind": kind, "family": family, "rows": rows, "cols": cols,
                "depth": 1 if family == "qft" else rng.randint(4, 14),
                "fusion": fusion, "max_k": rng.randint(3, 6),
                "precision": rng.choice(("fp32_valu", "fp32_valu", "fp32_mfma", "bf16x3", "fp16x3")),
                "graph": rng.random() < 0.3}
    if kind == "batch":
        lo = rng.randint(6, 14)
        return {"kind": kind, "count": rng.randint(5, 60), "n_min": lo, "n_max": lo + rng.randint(0, 8),
                "layers": rng.randint(2, 8), "max_k": rng.randint(2, 5), "fusion": rng.choice(("block", "greedy"))}
    if kind == "pauli":
        rows, cols = rng.choice(((1, 9), (3, 4), (2, 7), (3, 5), (4, 4), (3, 6), (4, 6), (5, 5), (2, 13), (1, 27)))
        return {"kind": kind, "rows": rows, "cols": cols}
    if kind == "reads":
        n = rng.randint(10, 28)
        return {"kind": kind, "n": n, "measured": rng.randint(1, min(10, n)),
                "shots": int(math.exp(rng.uniform(math.log(100), math.log(200000))))}
    return {"kind": "train", "samples": int(math.exp(rng.uniform(math.log(300), math.log(7200)))),
            "epochs": rng.randint(1, 20)}


# ---------------------------------------------------------------- inputs
def _random_state(n, seed):
    """A normalised Gaussian complex64 state on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    v = torch.randn(1 << n, dtype=torch.complex64, device="cuda", generator=g)
    v *= 1.0 / float(torch.linalg.vector_norm(torch.view_as_real(v), dtype=torch.float64))
    return v


def _gate_of(case, seed):
    """The gate of a `gate` case: Haar-random; the qubits belong to the case."""
    n, k, nc = case["n"], case["k"], case["controls"]
    pick = np.random.Generator(np.random.PCG64(1000 * n + 10 * k + nc))
    if case["low"]:  # targets from the low end, where a gather splits cache lines
        pool = list(pick.permutation(min(n, k + nc + 3)))
    else:
        pool = list(pick.permutation(n))
    qubits = tuple(int(q) for q in pool[:k])
    controls = tuple(int(q) for q in pool[k:k + nc])
    return qubits, controls, C.haar_unitary(k, np.random.Generator(np.random.PCG64(seed)))


def _qubits(case):
    return case["rows"] * case["cols"]


def _circuit_of(case, seed):
    if case["family"] == "grid":
        return C.grid_circuit(case["rows"], case["cols"], case["depth"], seed=seed)
    if case["family"] == "qv":
        return C.quantum_volume_circuit(_qubits(case), case["depth"], seed=seed)
    return C.qft_like_circuit(_qubits(case))


def _start_of(case, seed):
    return C.qft_input_basis(_qubits(case), seed) if case["family"] == "qft" else 0


def _batch_of(case, seed):
    span = case["n_max"] - case["n_min"] + 1
    ns = [case["n_min"] + (5 * i) % span for i in range(case["count"])]
    rng = np.random.Generator(np.random.PCG64(seed))
    return ns, [C.ansatz_circuit(n, rng.uniform(0.0, 2 * np.pi, size=(case["layers"], n, 2))) for n in ns]


def _ising(case):
    n = _qubits(case)
    zz = [e for p in range(4) for e in C.grid_couplers(case["rows"], case["cols"], p)]
    x = [0] * len(zz) + [1 << q for q in range(n)]
    z = [(1 << a) | (1 << b) for a, b in zz] + [0] * n
    return np.array(x, dtype=np.uint64), np.array(z, dtype=np.uint64)


def _corpus(samples, seed):
    """Features and targets shaped like the cost model's timing corpus."""
    rng = np.random.Generator(np.random.PCG64(seed))
    x = np.zeros((samples, sv.SV_COST_FEATURES), dtype=np.float32)
    for i in range(samples):
        n, k = int(rng.choice((26, 28, 30))), int(rng.integers(1, 7))
        x[i] = sv.sv_cost_features(k, rng.permutation(n)[:k].tolist(), n, int(rng.integers(0, 4)))
    y = (-5.5 + 0.8 * x[:, 0] + 0.1 * x[:, 2:36].sum(1) + 0.1 * rng.standard_normal(samples)).astype(np.float32)
    return torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "gate":
        s["qubits"], s["controls"], s["matrix"] = _gate_of(case, seed)
        s["state"] = sv.State(case["n"])
        s["state"].buf.copy_(_random_state(case["n"], seed))
    elif kind in ("circuit", "step"):
        s["gates"] = sv.GateArray(_circuit_of(case, seed))
        s["start"] = _start_of(case, seed)
        s["state"] = sv.State(_qubits(case))
    elif kind == "batch":
        ns, circs = _batch_of(case, seed)
        s["states"] = [sv.State(n) for n in ns]
        # marshalled once, as the benchmark's batched workload does
        s["arrays"] = [sv.GateArray(c) for c in circs]
        count = len(ns)
        s["handles"] = (ctypes.c_void_p * count)(*[t.h for t in s["states"]])
        s["circuits"] = (ctypes.POINTER(sv.sv_gate) * count)(*[a.ptr for a in s["arrays"]])
        s["lengths"] = (ctypes.c_size_t * count)(*[a.n for a in s["arrays"]])
        s["opts"] = sv.make_opts(max_k=case["max_k"], fusion=case["fusion"])
    elif kind == "pauli":
        n = _qubits(case)
        s["x"], s["z"] = _ising(case)
        s["state"] = sv.State(n)
        s["state"].buf.copy_(_random_state(n, seed))
    elif kind == "reads":
        s["state"] = sv.State(case["n"])
        s["state"].buf.copy_(_random_state(case["n"], seed))
        s["measured"] = tuple(range(0, case["n"], max(1, case["n"] // case["measured"])))[:case["measured"]]
        s["uniforms"] = C.uniforms(case["shots"], seed)
    else:
        s["x"], s["y"] = _corpus(case["samples"], seed)
        s["model"] = sv.Mlp(seed=seed)
        s["params"] = s["model"].get_params()
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "gate":
        if s["controls"]:
            s["state"].apply_controlled_gate(s["qubits"], s["matrix"], s["controls"])
        else:
            s["state"].apply_gate(s["qubits"], s["matrix"])
        return s["state"].buf
    if kind in ("circuit", "step"):
        st = s["state"]
        st.set_basis(s["start"])
        st.apply_circuit(s["gates"], max_k=case["max_k"], fusion=case["fusion"], precision=case["precision"],
                         use_graph=case["graph"])
        if kind == "circuit":
            return st.buf
        return {"state": st.buf, "norm": st.norm(), "head": st.read(0, READ_BACK)}
    if kind == "batch":
        for t in s["states"]:
            t.set_basis(0)
        rc = sv.lib().sv_batch_run(s["handles"], s["circuits"], s["lengths"], len(s["states"]),
                                   ctypes.byref(s["opts"]), None)
        if rc != sv.SV_OK:
            raise sv.SvError(rc, sv.lib().sv_last_error().decode())
        return [t.buf for t in s["states"]]
    if kind == "pauli":
        return s["state"].expect_pauli(s["x"], s["z"])
    if kind == "reads":
        st = s["state"]
        return {"norm": st.norm(), "marginal": st.marginal_probs(s["measured"]),
                "samples": st.sample(s["uniforms"]).astype(np.int64)}
    s["model"].set_params(s["params"])
    loss = s["model"].train(s["x"], s["y"], epochs=case["epochs"], lr=3e-3)
    return {"loss": loss, "params": s["model"].get_params()}


# ------------------------------------------------------ what a pass has to do
def work(case):
    """State bytes read and written once; the flops of the gates one by one
    (a diagonal gate is one complex product per amplitude)."""
    kind = case["kind"]

    def gate_flops(n, gates):
        total = 0.0
        for g in gates:
            dense = np.count_nonzero(g.matrix - np.diag(np.diag(g.matrix)))
            total += 2.0 ** n * (8.0 * 2 ** g.k - 2.0 if dense else 6.0)
        return total

    if kind == "gate":
        amps = 2.0 ** (case["n"] - case["controls"])
        return {"bytes": 16.0 * amps, "flops": amps * (8.0 * 2 ** case["k"] - 2.0)}
    if kind in ("circuit", "step"):
        n = _qubits(case)
        return {"bytes": 16.0 * 2 ** n, "flops": gate_flops(n, _circuit_of(case, 0))}
    if kind == "batch":
        ns, circs = _batch_of(case, 0)
        return {"bytes": sum(16.0 * 2 ** n for n in ns), "flops": sum(gate_flops(n, c) for n, c in zip(ns, circs))}
    if kind == "pauli":
        return {"bytes": 8.0 * 2 ** _qubits(case), "flops": 8.0 * 2 ** _qubits(case) * len(_ising(case)[0])}
    if kind == "reads":
        return {"bytes": 8.0 * 2 ** case["n"], "flops": 3 * 4.0 * 2 ** case["n"]}
    params = 40 * 64 + 64 * 64 + 64
    return {"bytes": 164.0 * case["samples"], "flops": 6.0 * params * case["samples"] * case["epochs"]}


# -------------------------------------------------- the same in 64 bits
def _apply(psi, n, qubits, matrix, controls=()):
    """One gate on a complex128 state, in place (qubit q is bit q)."""
    k = len(qubits)
    view = psi.view((2,) * n)
    at = [slice(None)] * n
    for c in controls:
        at[n - 1 - c] = 1
    parts = []
    for l in range(1 << k):
        for j, q in enumerate(qubits):
            at[n - 1 - q] = (l >> j) & 1
        parts.append(view[tuple(at)])
    m = np.asarray(matrix, dtype=np.complex128)
    if not np.count_nonzero(m - np.diag(np.diag(m))):
        for l in range(1 << k):
            if m[l, l] != 1.0:
                parts[l].mul_(complex(m[l, l]))
        return
    old = [p.clone() for p in parts]
    for r in range(1 << k):
        parts[r].mul_(complex(m[r, r]))
        for c in range(1 << k):
            if c != r and m[r, c] != 0.0:
                parts[r].add_(old[c], alpha=complex(m[r, c]))


def _simulate(n, gates, start=0):
    psi = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    psi[start] = 1.0
    for g in gates:
        _apply(psi, n, g.qubits, g.matrix, g.controls)
    return psi


def _adam64(case, seed):
    """The training loop in float64: 40 -> 64 -> 64 -> 1, mean squared error."""
    x, y = (t.double() for t in _corpus(case["samples"], seed))
    m = sv.Mlp(seed=seed)
    flat = torch.tensor(m.get_params(), device="cuda").double()
    m.free()
    f, w = sv.SV_COST_FEATURES, 64
    sizes = [(w, f), (w,), (w, w), (w,), (1, w), (1,)]

    def loss_of(p):
        t, parts = 0, []
        for shape in sizes:
            parts.append(p[t:t + math.prod(shape)].reshape(shape))
            t += math.prod(shape)
        w1, b1, w2, b2, w3, b3 = parts
        h = torch.relu(torch.relu(x @ w1.T + b1) @ w2.T + b2)
        return ((h @ w3.T + b3)[:, 0] - y).square().mean()

    mom, var = torch.zeros_like(flat), torch.zeros_like(flat)
    for step in range(1, case["epochs"] + 1):
        p = flat.requires_grad_(True)
        g, = torch.autograd.grad(loss_of(p), p)
        mom = 0.9 * mom + 0.1 * g
        var = 0.999 * var + 0.001 * g * g
        flat = (p - 3e-3 * (mom / (1 - 0.9 ** step)) / ((var / (1 - 0.999 ** step)).sqrt() + 1e-8)).detach()
    return {"loss": float(loss_of(flat)), "params": flat}


def exact(case, seed):
    kind = case["kind"]
    if kind == "gate":
        psi = _random_state(case["n"], seed).to(torch.complex128)
        qubits, controls, matrix = _gate_of(case, seed)
        _apply(psi, case["n"], qubits, matrix, controls)
        return psi
    if kind == "circuit":
        return _simulate(_qubits(case), _circuit_of(case, seed), _start_of(case, seed))
    if kind == "step":
        return None  # a 30-qubit complex128 run takes longer than the case is worth
    if kind == "batch":
        ns, circs = _batch_of(case, seed)
        return [_simulate(n, c) for n, c in zip(ns, circs)]
    if kind == "pauli":
        n = _qubits(case)
        psi = _random_state(n, seed).to(torch.complex128)
        p = psi.abs().square()
        out = []
        for x, z in zip(*_ising(case)):
            if x:
                v = psi.view(-1, 2, int(x))
                out.append(2.0 * float((v[:, 0].conj() * v[:, 1]).real.sum()))
            else:
                a, b = (i for i in range(n) if (int(z) >> i) & 1)
                v = p.view(-1, 2, 1 << (b - a - 1), 2, 1 << a)
                out.append(float((v[:, 0, :, 0] + v[:, 1, :, 1] - v[:, 0, :, 1] - v[:, 1, :, 0]).sum()))
        return np.array(out)
    if kind == "reads":
        n, m = case["n"], case["measured"]
        p = _random_state(n, seed).to(torch.complex128).abs().square()
        measured = tuple(range(0, n, max(1, n // m)))[:m]
        index = torch.arange(1 << n, device="cuda")
        outcome = torch.zeros_like(index)
        for j, q in enumerate(measured):
            outcome |= ((index >> q) & 1) << j
        marginal = torch.bincount(outcome, weights=p, minlength=1 << m)
        return {"norm": float(p.sum()), "marginal": marginal.cpu().numpy(), "samples": None}
    return _adam64(case, seed)
