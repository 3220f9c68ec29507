"""Gates as rotations in the LDS circuits (batch jobs and stages), at the
angles where the form changes (45, 90, 180 degrees and just beside them), with
the scales that the two-step form leaves on the registers in front of every
other kind of gate, and many of them on one qubit; and measurements of staged
jobs by chunks.  Against the oracle.

Tolerance: a gate changes an amplitude by at most 4 u of the state's norm (u =
2^-53 or 2^-24: three steps and a rounded coefficient), and a pass by 2 u more
(its scales), fewer than the gates: 6 u per gate, over the 2-norm and so over
the largest difference, plus 1e-13 for the oracle's own rounding."""
import math

import numpy as np
import pytest

import oracle
import workloads as W
from workloads.circuits import rng_for

pytestmark = pytest.mark.gpu

QUARTER = math.pi / 2   # a rotation's angle is half the gate's parameter: 45 degrees
ANGLES = [0.0, QUARTER, -QUARTER, QUARTER - 1e-6, QUARTER + 1e-6, math.pi, -math.pi, math.pi - 1e-6, math.pi + 1e-6,
          3 * QUARTER, -3 * QUARTER + 1e-6, 2 * math.pi, 2 * math.pi - 1e-6, 3 * math.pi, 4 * math.pi, 0.3, -2.0, 5.0]


def _tol(dtype, gates):
    return 6 * gates * (2.0 ** -53 if dtype == "c128" else 2.0 ** -24) + 1e-13


def _edge_angles(n, seed):
    """Every rotation at every angle, on each other's heels."""
    rng = rng_for(seed)
    ops = [W.add_qubits(n)] + [W.gate("RY", [q], params=(0.4 + q,)) for q in range(n)]
    for k, t in enumerate(ANGLES):
        q = [int(x) for x in rng.permutation(n)]
        ops += [W.gate(("RX", "RY", "RZ")[(k + j) % 3], [q[j % n]], params=(t,)) for j in range(3)]
        if n > 1:
            ops += [W.gate("RZZ", [q[0], q[1]], params=(t,)), W.gate("X", [q[0]], controls=[q[1]])]
        ops.append(W.gate(("H", "X", "Y", "T")[k % 4], [q[-1]]))
    return W.Circuit(ops, label=f"angles_n{n}")


def _scaled(n, seed):
    """Scales of both kinds (imaginary parts, slots) in front of masked gates,
    flips, phases and swaps, all in one pass; cbit conditions."""
    rng = rng_for(seed)
    ops = [W.add_qubits(n), W.add_cbits(2), W.gate("H", [0]), W.measure(0, cbit=0, u=0.3), W.gate("RX", [0], params=(1.1,))]
    for k in range(10):
        a, b, c = [int(x) for x in rng.permutation(n)[:3]]
        ops += [W.gate("RZ", [a], params=(0.7 + k,)), W.gate("RY", [b], params=(0.5 + k,)),
                W.gate("RX", [a], params=(0.9 - k,)), W.gate("H", [c])]
        ops.append([W.gate("RX", [b], controls=[a], params=(0.8,)), W.gate("RY", [a], controls=[b], params=(1.9,)),
                    W.gate("X", [b], controls=[a, c]), W.gate("H", [a], controls=[c]), W.gate("T", [a]),
                    W.gate("CPHASE", [a, b], params=(0.6,)), W.gate("SWAP", [a, b], controls=[c]),
                    W.gate("RX", [c], conds=[(0, k % 2)], params=(1.3,)), W.gate("RZ", [b], controls=[c], params=(2.2,)),
                    W.gate("Y", [a], controls=[b])][k])
    return W.Circuit(ops, label=f"scaled_n{n}")


def _many_on_one(n):
    """The largest scales a pass can reach: two-step rotations of one slot and
    of the imaginary parts, just below 45 degrees, as many as a pass holds."""
    t = QUARTER - 1e-3
    ops = [W.add_qubits(n), W.gate("H", [0])]
    for k in range(48):
        ops.append(W.gate("RZ" if k % 2 else "RY", [0], params=(t if k % 3 else -t,)))
    return W.Circuit(ops, label=f"many_n{n}")


def _check(circ, got, dtype):
    ref, _, recs = oracle.run(circ)
    assert all(abs(r.u - r.P0) > 1e-6 for r in recs)
    d = float(np.max(np.abs(got.astype(np.complex128) - ref)))
    tol = _tol(dtype, len(circ.gate_ops()))
    print(f"[gpu-rotations] {circ.label} {dtype}: max|d| = {d:.2e} (tol {tol:.2e})", flush=True)
    assert d <= tol


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_batch_jobs(dtype):
    """One chunk of 1 to 13 (14) qubits, and the smallest staged jobs."""
    import paper_1908_07187_amd as qk
    top = 13 if dtype == "c128" else 14
    circs = [_edge_angles(n, n) for n in (1, 2, 3, 4, 5, 8, top - 1, top, top + 1)]
    circs += [_scaled(n, n) for n in (3, 4, 5, 9, top, top + 1)] + [_many_on_one(n) for n in (1, 4, 6, top + 1)]
    b = qk.Batch(dtype)
    ids = [qk.add_circuit(b, c) for c in circs]
    b.run()
    b.sync()
    for c, j in zip(circs, ids):
        _check(c, b.state(j), dtype)
    b.close()


@pytest.mark.parametrize("n", [13, 14, 16])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_stages(n, dtype):
    import paper_1908_07187_amd as qk
    for c in (_edge_angles(n, 3), _scaled(n, 5), _many_on_one(n)):
        s = qk.Sim(dtype)
        s.set_tuning("stages", 1)
        qk.Program(c).run(s)
        _check(c, s.state(), dtype)
        s.close()


@pytest.mark.parametrize("dtype,n", [("c128", 14), ("c128", 20), ("c128", 21), ("c64", 15), ("c64", 21), ("c64", 22)])
def test_staged_measurement(dtype, n):
    """Measurements of a staged job, one after another, of the lowest and the
    highest qubit: 2 chunks of sums, 256 of one stage chunk each, and 256 of
    two; cbits steer later gates.  The cbits of every job are read back, also
    after a job with more of them was added and on a second run."""
    import paper_1908_07187_amd as qk

    def circuit(k):
        ops = [W.add_qubits(n), W.add_cbits(k)] + [W.gate("RY", [q], params=(0.3 + 0.1 * q,)) for q in range(n)]
        for j, q in enumerate([0, n - 1, n // 2][:k]):
            ops += [W.measure(q, cbit=j, u=(0.9, 0.05, 0.7)[j]), W.gate("RX", [(q + 1) % n], conds=[(j, 1)], params=(1.0,)),
                    W.gate("X", [q], controls=[(q + 2) % n])]
        return W.Circuit(ops, label=f"measured_n{n}_k{k}")

    b = qk.Batch(dtype)
    circs = [circuit(2)]
    ids = [qk.add_circuit(b, circs[0])]
    b.run()
    assert list(b.cbits(ids[0])) == list(oracle.run(circs[0])[1])
    circs.append(circuit(3))
    ids.append(qk.add_circuit(b, circs[1]))
    for _ in range(2):
        b.run()
        b.sync()
        for c, j in zip(circs, ids):
            assert list(b.cbits(j)) == list(oracle.run(c)[1])
            _check(c, b.state(j), dtype)
    b.close()
