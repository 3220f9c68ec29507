"""Cases that time this engine's public entry points on the work its users have it do.

Sizes and recipes are the repository's own: the layered random circuit, the QFT, iterative
phase estimation and Shor recipes of ``workloads``, the job sizes of the batch and serving
benchmarks, and the gate classes of the tests.  ``exact`` recomputes a case's outputs in
64 bits with plain torch, from the circuit description alone.
"""
import ctypes as C
import math

import numpy as np
import torch

import paper_1908_07187_amd as qk
import workloads as W
from paper_1908_07187_amd import autotune
from paper_1908_07187_amd.batch import op_array
from workloads.circuits import big_endian_bits, rng_for

AMP = {"c64": 8, "c128": 16}


def listed():
    return [
        # A small register worked on interactively: every gate its own call, default settings,
        # the state read back to the host.  Latency and launch counts.
        {"name": "eager_small", "kind": "circuit", "form": "layers", "mode": "default", "n": 8, "layers": 10,
         "dtype": "c128"},
        # A large register gate by gate with default settings: one layer of the depth-40 benchmark circuit's
        # recipe, each gate a sweep of 4 GiB.
        {"name": "eager_large", "kind": "circuit", "form": "layers", "mode": "default", "n": 28, "layers": 1,
         "dtype": "c128"},
        # Mid-size requests of the serving mix: an op list in one call on a simulator set up by the autotuner.
        {"name": "tuned_mid", "kind": "circuit", "form": "layers", "mode": "tuned", "n": 21, "layers": 20,
         "dtype": "c128"},
        # The benchmark circuit's recipe at large sizes, set up by the autotuner, both precisions.
        {"name": "tuned_large_c128", "kind": "circuit", "form": "layers", "mode": "tuned", "n": 28, "layers": 8,
         "dtype": "c128"},
        {"name": "tuned_large_c64", "kind": "circuit", "form": "layers", "mode": "tuned", "n": 28, "layers": 8,
         "dtype": "c64"},
        # The 26-qubit QFT and its inverse with default settings, on a product state.
        {"name": "qft", "kind": "circuit", "form": "qft", "mode": "default", "n": 26, "layers": 1, "dtype": "c128"},
        # Many equal small circuits in one launch (parameter sweeps, shot ensembles).
        {"name": "batch_small", "kind": "batch", "jobs": 2048, "n_lo": 12, "n_hi": 12, "layers": 20, "measure": False,
         "dtype": "c128"},
        # Ragged mid-size jobs in one launch, a third of them with a measurement that steers a later gate.
        {"name": "batch_mid", "kind": "batch", "jobs": 96, "n_lo": 8, "n_hi": 20, "layers": 20, "measure": True,
         "dtype": "c64"},
        # Iterative phase estimation as one captured graph, new uniforms for each run, cbits read back.
        {"name": "ipe_graph", "kind": "ipe", "m": 20, "dtype": "c128"},
        # User-defined gates: unitaries on 1 to 6 qubits, with and without a control, a permutation table and a
        # modular multiplication.
        {"name": "user_gates", "kind": "user", "n": 25, "rounds": 2, "dtype": "c64"},
        # Deferred measurement: many shots and a 10-qubit distribution of a dense random state.
        {"name": "sample", "kind": "sample", "n": 26, "shots": 1 << 18, "dtype": "c128"},
        # The conventional Shor circuit on the sparse engine (27 qubits, up to 2^18 entries).
        {"name": "shor_sparse", "kind": "sparse", "N": 509, "dtype": "c128"},
    ]


def draw(rng):
    kind = rng.choice(["circuit", "circuit", "circuit", "circuit", "batch", "batch", "ipe", "user", "sample", "sparse"])
    dtype = rng.choice(["c64", "c128"])
    if kind == "circuit":
        mode = rng.choice(["default", "tuned", "tuned"])
        form = rng.choice(["layers", "layers", "layers", "qft"])
        n = rng.randint(4, 27)
        top = 26 if mode == "tuned" else 12
        layers = 1 if form == "qft" else max(1, rng.randint(2, top) // (1 if n <= 24 else 4))
        return {"kind": kind, "form": form, "mode": mode, "n": min(n, 25) if form == "qft" else n, "layers": layers,
                "dtype": dtype}
    if kind == "batch":
        measure = rng.random() < 0.5
        lo = rng.randint(2, 12)
        hi = lo if not measure else rng.randint(max(lo, 10), 19)
        jobs = int(round(math.exp(rng.uniform(math.log(8), math.log(1500 if hi <= 12 else 64)))))
        return {"kind": kind, "jobs": jobs, "n_lo": lo, "n_hi": hi, "layers": rng.randint(4, 20), "measure": measure,
                "dtype": dtype}
    if kind == "ipe":
        return {"kind": kind, "m": rng.randint(6, 19), "dtype": dtype}
    if kind == "user":
        return {"kind": kind, "n": rng.randint(12, 24), "rounds": rng.randint(1, 2), "dtype": dtype}
    if kind == "sample":
        return {"kind": kind, "n": rng.randint(11, 25), "shots": int(round(math.exp(rng.uniform(math.log(100), math.log(200000))))),
                "dtype": dtype}
    return {"kind": "sparse", "N": rng.choice([21, 33, 55, 77, 105, 143, 187, 221, 253, 323, 391, 437]), "dtype": dtype}


# ---------------------------------------------------------------- circuits

def _circuit(case, seed):
    """The case's circuit (its add_* ops first, then gates and measurements)."""
    kind = case["kind"]
    if kind == "circuit":
        n = case["n"]
        if case["form"] == "layers":
            return W.c2_random_rzz(n=n, depth=case["layers"], seed=seed)
        th = rng_for(seed).uniform(0.2, math.pi - 0.2, n)
        bits = big_endian_bits(n)
        ops = [W.add_qubits(n)] + [W.gate("RY", [q], params=(float(th[q]),)) for q in range(n)]
        ops += W.qft_ops(bits)
        # phases between the transforms, so that the inverse does not undo the first one
        ops += [W.gate("RZ", [q], params=(float(th[q]),)) for q in range(n)]
        return W.Circuit(ops + W.qft_ops(bits, inverse=True), seed=seed)
    if kind == "ipe":
        return W.c3_ipe(m=case["m"], seed=seed)
    if kind == "user":
        return _user_circuit(case["n"], case["rounds"], seed)
    raise KeyError(kind)


def _user_circuit(n, rounds, seed):
    rng = rng_for(seed)
    ops, user = [W.add_qubits(n)] + [W.gate("H", [q]) for q in range(n)], {}

    def some(k):
        return [int(q) for q in rng.permutation(n)[:k]]

    for r in range(rounds):
        for k in range(1, 7):
            key = f"U{r}_{k}"
            user[key] = {"kind": "matrix", "k": k, "matrix": W.random_unitary(k, rng)}
            q = some(k + 1)
            ops.append(W.gate(key, q[:k], controls=q[k:] if (k + r) % 3 == 0 else ()))
        user[f"P{r}"] = {"kind": "table", "k": 10, "table": rng.permutation(1 << 10).astype(np.uint64)}
        ops.append(W.gate(f"P{r}", some(10)))
        user[f"M{r}"] = {"kind": "modmul", "k": 9, "a": 2, "N": 2 * int(rng.integers(100, 250)) + 1}
        q = some(10)
        ops.append(W.gate(f"M{r}", q[:9], controls=q[9:], params=(float(rng.integers(0, 4)),)))
    return W.Circuit(ops, user_gates=user, seed=seed)


def _jobs(case, seed):
    """The circuits of a batch."""
    rng, sizes = rng_for(seed), rng_for(case["jobs"])   # the sizes are the case's own, the gates the seed's
    out = []
    for j in range(case["jobs"]):
        if case["measure"]:
            n = int(sizes.integers(case["n_lo"], case["n_hi"] + 1))
            depth = 2 + int(sizes.integers(case["layers"] // 2, case["layers"] + 1))
            c, _ = W.c4_job(rng, n_range=(n, n), depth_range=(depth, depth), p_measure=1.0 if j % 3 == 0 else 0.0)
        else:
            c = W.c0_random_layers(n=case["n_lo"], layers=case["layers"], seed=int(rng.integers(1 << 30)))
        out.append(c)
    return out


def _body(circ):
    return W.Circuit([o for o in circ.ops if o.kind in ("gate", "measure")], user_gates=circ.user_gates)


def _view(sim, dtype):
    """The simulator's state as a device tensor (no copy)."""
    ptr, nbytes = sim.state_ptr()
    return _device_view(ptr, nbytes, dtype, sim)


class _Memory:
    """Device memory as torch.as_tensor takes it; the owner lives as long as the tensor."""

    def __init__(self, ptr, nbytes, dtype, owner):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (nbytes // AMP[dtype],), "typestr": "<c8" if dtype == "c64" else "<c16",
                                         "data": (ptr, False), "version": 3}


def _device_view(ptr, nbytes, dtype, owner):
    return torch.as_tensor(_Memory(ptr, nbytes, dtype, owner), device="cuda")


# ---------------------------------------------------------------- prepare and run

def prepare(case, seed):
    kind, dtype = case["kind"], case["dtype"]
    if kind == "batch":
        b, jobs = qk.Batch(dtype), _jobs(case, seed)
        for c in jobs:
            b.add(c.n_qubits, c.n_cbits, *op_array(c))
        measured = [j for j, c in enumerate(jobs) if any(o.kind == "measure" for o in c.ops)]
        return {"kind": kind, "batch": b, "dtype": dtype, "measured": measured}
    if kind == "sparse":
        N = case["N"]
        circ = W.shor_3nx1(N, 2, measure_work=True, seed=seed, tables=False)
        return {"kind": kind, "prog": qk.Program(circ), "dtype": dtype, "cap": 1 << (N * N - 1).bit_length(),
                "u": rng_for(seed).random(64), "ctrl": list(range(N.bit_length(), circ.n_qubits))}
    if kind == "sample":
        n = case["n"]
        g = torch.Generator(device="cuda").manual_seed(seed)
        sim = qk.Sim(dtype)
        sim.add_qubits(n)
        sim.set_state(_random_state(n, dtype, seed).cpu().numpy())
        return {"kind": kind, "sim": sim, "n": n, "shots": case["shots"],
                "u": torch.rand(case["shots"], dtype=torch.float64, device="cuda", generator=g),
                "out": torch.zeros(case["shots"], dtype=torch.int64, device="cuda"),
                "qubits": _sample_qubits(n, seed)}
    circ = _circuit(case, seed)
    body = _body(circ)
    if kind == "ipe":
        # capture takes a stream of its own; each run draws with the uniforms on the device
        sim = qk.Sim(dtype, stream=torch.cuda.Stream())
        sim.add_qubits(circ.n_qubits)
        sim.add_cbits(circ.n_cbits)
        prog = qk.Program(body)
        ids = prog.define_gates(sim)
        u = torch.tensor([o.u for o in circ.ops if o.kind == "measure"], dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        sim.capture_begin()
        sim.reset()
        prog.run(sim, d_uniforms=u.data_ptr(), ids=ids)
        return {"kind": kind, "sim": sim, "graph": sim.capture_end(), "u": u, "dtype": dtype}
    sim = qk.Sim(dtype)
    mode = case.get("mode", "default")
    if mode == "tuned":
        autotune.apply(sim, circ.n_qubits, dtype)
    sim.add_qubits(circ.n_qubits)
    st = {"kind": kind, "sim": sim, "dtype": dtype, "mode": mode, "host": circ.n_qubits <= 12}
    if mode == "tuned":
        st["ops"] = op_array(body)
    else:
        st["prog"] = qk.Program(body)
        st["ids"] = st["prog"].define_gates(sim)
    return st


def run(state):
    kind, dtype = state["kind"], state.get("dtype")
    if kind == "batch":
        b = state["batch"]
        b.run()
        out = {"states": _device_view(_batch_ptr(b), b.sizes()[0], dtype, b)}
        if state["measured"]:
            out["cbits"] = np.concatenate([b.cbits(j) for j in state["measured"]])
        return out
    if kind == "sparse":
        sim = qk.Sim(dtype, sparse=state["cap"])
        state["prog"].run(sim)
        shots = sim.sample(state["u"], state["ctrl"])
        idx, amp = sim.entries()
        sim.close()
        return {"shots": shots.astype(np.int64), "index": idx.astype(np.int64), "amplitude": amp}
    sim = state["sim"]
    if kind == "sample":
        sim.sample_dev(state["u"].data_ptr(), state["shots"], state["out"].data_ptr())
        return {"shots": state["out"], "distribution": sim.probabilities(state["qubits"])}
    if kind == "ipe":
        state["graph"].launch()
        return {"cbits": sim.read_cbits(), "state": _view(sim, dtype)}
    sim.reset()
    if state["mode"] == "tuned":
        sim.apply_ops(*state["ops"])
    else:
        state["prog"].run(sim, ids=state["ids"])
    return sim.state() if state["host"] else _view(sim, dtype)


def _batch_ptr(b):
    """The device address of the batch's states (the first job's starts the buffer)."""
    p, nbytes = C.c_void_p(), C.c_size_t()
    if b.lib.qk_batch_state_ptr(b.h, 0, C.byref(p), C.byref(nbytes)) != qk.qk.QK_OK:
        raise RuntimeError("qk_batch_state_ptr")
    return int(p.value)


def _random_state(n, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    v = torch.randn(1 << n, dtype=torch.complex128, device="cuda", generator=g)
    v /= torch.linalg.vector_norm(v)
    return v.to(torch.complex64) if dtype == "c64" else v


def _sample_qubits(n, seed):
    return [int(q) for q in rng_for(seed).permutation(n)[:10]]


# ---------------------------------------------------------------- work

def _gate_flops(op, n, user):
    size = 2.0 ** (n - len(op.controls))
    if op.name in user:
        return 8.0 * size * (1 << user[op.name]["k"]) if user[op.name]["kind"] == "matrix" else 0.0
    if op.name in ("X", "SWAP"):
        return 0.0
    if op.name in ("CPHASE", "PHASE", "S", "T", "SDG", "TDG", "Z"):
        return 6.0 * size / 2 ** len(op.targets)
    if op.name in ("RZ", "RZZ"):
        return 6.0 * size
    return 6.0 * size if op.name in ("H", "RY", "RX", "Y") else 14.0 * size


def _circuit_work(circ, amp):
    n = circ.n_qubits
    flops = sum(_gate_flops(o, n, circ.user_gates) for o in circ.ops if o.kind == "gate")
    flops += sum(6.0 * 2 ** n for o in circ.ops if o.kind == "measure")
    return amp * 2.0 ** n, flops


def work(case):
    amp, kind = AMP[case["dtype"]], case["kind"]
    if kind == "batch":
        done = [_circuit_work(c, amp) for c in _jobs(case, 1)[:256]]
        scale = case["jobs"] / len(done)
        return {"bytes": scale * sum(b for b, _ in done), "flops": scale * sum(f for _, f in done)}
    if kind == "sample":
        return {"bytes": 2.0 * amp * 2 ** case["n"] + 16.0 * case["shots"], "flops": 6.0 * 2 ** case["n"]}
    if kind == "sparse":
        entries = 2.0 ** (case["N"] ** 2 - 1).bit_length()
        return {"bytes": entries * (8 + amp), "flops": 10.0 * entries * (case["N"] ** 2 - 1).bit_length()}
    b, f = _circuit_work(_circuit(case, 1), amp)
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- exact values

def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        jobs = _jobs(case, seed)
        if not case["measure"]:
            return {"states": _equal_circuits(jobs).reshape(-1)}
        got = [_simulate(c) for c in jobs]
        return {"states": torch.cat([g[0] for g in got]), "cbits": None}
    if kind == "sparse":
        return None   # entries that cancel to rounding have no exact position in the list
    if kind == "sample":
        p = _random_state(case["n"], case["dtype"], seed).to(torch.complex128)
        p = p.real.square() + p.imag.square()
        i = torch.arange(p.numel(), device="cuda")
        m = sum(((i >> q) & 1) << j for j, q in enumerate(_sample_qubits(case["n"], seed)))
        return {"shots": None, "distribution": torch.bincount(m, weights=p, minlength=1 << 10) / p.sum()}
    psi, _ = _simulate(_circuit(case, seed))
    return {"cbits": None, "state": psi} if kind == "ipe" else psi


def _matrix(op, user):
    """The gate's matrix over its targets (bit j of an index is targets[j]), complex128."""
    if op.name in user:
        return np.asarray(user[op.name]["matrix"], dtype=np.complex128)
    a = op.params[0] if op.params else 0.0
    c, s, e = math.cos(a / 2), math.sin(a / 2), complex(math.cos(a / 2), -math.sin(a / 2))
    p = complex(math.cos(a), math.sin(a))
    r, t = math.sqrt(0.5), complex(math.sqrt(0.5), math.sqrt(0.5))
    diag = {"Z": [1, -1], "S": [1, 1j], "SDG": [1, -1j], "T": [1, t], "TDG": [1, t.conjugate()], "PHASE": [1, p],
            "RZ": [e, e.conjugate()], "CPHASE": [1, 1, 1, p], "RZZ": [e, e.conjugate(), e.conjugate(), e]}
    if op.name in diag:
        return np.diag(np.array(diag[op.name], dtype=np.complex128))
    full = {"H": [[r, r], [r, -r]], "X": [[0, 1], [1, 0]], "Y": [[0, -1j], [1j, 0]], "RX": [[c, -1j * s], [-1j * s, c]],
            "RY": [[c, -s], [s, c]], "SWAP": [[1, 0, 0, 0], [0, 0, 1, 0], [0, 1, 0, 0], [0, 0, 0, 1]]}
    return np.array(full[op.name], dtype=np.complex128)


def _pieces(psi, n, targets, controls):
    """Views of psi, one per value of the target bits (targets[0] lowest), where every control bit is 1."""
    qs = sorted(list(targets) + list(controls), reverse=True)
    shape, top = [], n
    for q in qs:
        shape += [1 << (top - 1 - q), 2]
        top = q
    v = psi.view(shape + [1 << top])
    out = []
    for r in range(1 << len(targets)):
        bit = {q: (r >> j) & 1 for j, q in enumerate(targets)}
        w = v
        for at in range(len(qs) - 1, -1, -1):   # the last dimension first, so earlier ones keep their places
            w = w.select(2 * at + 1, bit.get(qs[at], 1))
        out.append(w)
    return out


def _permute(psi, n, op, g):
    """The state after a permutation gate."""
    i = torch.arange(psi.numel(), device=psi.device)
    x = sum(((i >> q) & 1) << j for j, q in enumerate(op.targets))
    j = int(op.params[0]) if op.params else 0
    if g["kind"] == "table":
        y = torch.from_numpy(np.asarray(g["table"]).astype(np.int64)).to(psi.device)[x]
    elif g["kind"] == "modmul":
        y = torch.where(x < g["N"], x * pow(g["a"], 1 << j, g["N"]) % g["N"], x)
    else:
        a, b, mod = g["a"], g["b"], 1 << g["k"]
        for _ in range(j):
            a, b = a * a % mod, (a * b + b) % mod
        y = (x * a + b) % mod
    to = i
    for k, q in enumerate(op.targets):
        to = (to & ~(1 << q)) | (((y >> k) & 1) << q)
    for c in op.controls:
        to = torch.where(((i >> c) & 1) == 1, to, i)
    out = torch.empty_like(psi)
    out[to] = psi
    return out


def _simulate(circ):
    """(final state, cbits) of a circuit from |0...0>, in complex128."""
    n = circ.n_qubits
    psi = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    psi[0] = 1
    cbits = [0] * circ.n_cbits
    for op in circ.ops:
        if op.kind == "measure":
            zero, one = _pieces(psi, n, [op.qubit], [])
            p = [float((w.real.square() + w.imag.square()).sum()) for w in (zero, one)]
            got = 0 if op.u < p[0] / (p[0] + p[1]) else 1
            (one if got == 0 else zero).zero_()
            (zero, one)[got].mul_(1.0 / math.sqrt(p[got]))
            if op.cbit >= 0:
                cbits[op.cbit] = got
        elif op.kind == "gate" and all(cbits[c] == v for c, v in op.conds):
            g = circ.user_gates.get(op.name)
            if g is not None and g["kind"] != "matrix":
                psi = _permute(psi, n, op, g)
                continue
            m, parts = _matrix(op, circ.user_gates), _pieces(psi, n, op.targets, op.controls)
            if np.count_nonzero(m - np.diag(np.diag(m))) == 0:
                for r, w in enumerate(parts):
                    if m[r, r] != 1:
                        w.mul_(complex(m[r, r]))
                continue
            if len(parts) <= 4:
                new = [sum(complex(m[r, c]) * parts[c] for c in range(len(parts)) if m[r, c] != 0) for r in range(len(parts))]
            else:
                new = torch.from_numpy(m).to(psi.device) @ torch.stack([w.reshape(-1) for w in parts])
            for w, x in zip(parts, new):
                w.copy_(x.view(w.shape))
    return psi, cbits


def _equal_circuits(jobs):
    """The final states of circuits that are alike but for angles, gate choices and qubits: (jobs, 2^n), complex128."""
    n, J = jobs[0].n_qubits, len(jobs)
    psi = torch.zeros(J, 1 << n, dtype=torch.complex128, device="cuda")
    psi[:, 0] = 1
    half = torch.arange(1 << (n - 1), device="cuda")[None, :]
    gates = [c.gate_ops() for c in jobs]
    for ops in zip(*gates):
        t = torch.tensor([o.targets[0] for o in ops], device="cuda")[:, None]
        c = torch.tensor([o.controls[0] if o.controls else -1 for o in ops], device="cuda")[:, None]
        m = torch.from_numpy(np.stack([_matrix(o, {}) for o in ops])).to("cuda")
        lo = ((half >> t) << (t + 1)) | (half & ((1 << t) - 1))
        hi = lo | (1 << t)
        a, b = psi.gather(1, lo), psi.gather(1, hi)
        on = (c < 0) | (((lo >> c.clamp(min=0)) & 1) == 1)
        psi.scatter_(1, lo, torch.where(on, m[:, 0, 0, None] * a + m[:, 0, 1, None] * b, a))
        psi.scatter_(1, hi, torch.where(on, m[:, 1, 0, None] * a + m[:, 1, 1, None] * b, b))
    return psi
