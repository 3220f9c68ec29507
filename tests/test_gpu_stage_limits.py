"""The stage queue ("stages") at the limits of what it takes: conditions past
the two that an op record holds, where such gates run as sweeps between the
stages.  Against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def _check(circ, dtype, got):
    """6 u per gate (two roundings and a rounded coefficient each, over the 2-norm), and 1e-13 for the oracle's own."""
    ref, cb, _ = oracle.run(circ)
    d = float(np.max(np.abs(got.astype(np.complex128) - ref)))
    tol = 6 * len(circ.gate_ops()) * (2.0 ** -53 if dtype == "c128" else 2.0 ** -24) + 1e-13
    print(f"[gpu-stage-limits] {circ.label} {dtype}: max|d| = {d:.2e} (tol {tol:.2e})", flush=True)
    assert d <= tol
    return list(cb)


def _conditioned(n):
    """Cbits 1, 0, 1, 0, ... by measurements of basis states, then gates with
    1 to 8 conditions that all hold, or all but the last or the first one."""
    ops = [W.add_qubits(n), W.add_cbits(8)]
    for c in range(8):
        ops += [W.gate("X", [c])] * (1 - c % 2) + [W.measure(c, cbit=c, u=0.5)]
    ops += [W.gate("RY", [q], params=(0.3 + 0.1 * q,)) for q in range(n)]
    for k in (1, 2, 3, 4, 5, 8):
        holds = [(c, 1 - c % 2) for c in range(k)]
        for j, conds in enumerate((holds, holds[:-1] + [(k - 1, k % 2 ^ 1)], [(0, 0)] + holds[1:])):
            q = (3 * k + j) % n
            ops += [W.gate("RX", [q], conds=conds, params=(0.7 + j,)), W.gate("H", [(q + 1) % n]),
                    W.gate("X", [(q + 2) % n], controls=[q], conds=conds),
                    W.gate("CPHASE", [q, (q + 4) % n], conds=conds, params=(0.4 + k,)), W.gate("RY", [q], params=(0.2,))]
    return W.Circuit(ops, label=f"conditions_n{n}")


@pytest.mark.parametrize("dtype,n", [("c128", 13), ("c64", 13), ("c128", 16), ("c64", 16)])
def test_any_number_of_conditions(dtype, n):
    import paper_1908_07187_amd as qk
    c = _conditioned(n)
    s = qk.Sim(dtype)
    s.set_tuning("stages", 1)
    qk.Program(c).run(s)
    got, cb = s.state(), list(s.read_cbits())
    s.close()
    assert cb == _check(c, dtype, got) == [1, 0] * 4


def _reference(circ):
    """The oracle's state.  (Its X multiplies by the matrix's zeros, so that one
    that is not finite reaches both of a pair: a last X is applied here.)"""
    last = circ.ops[-1]
    if last.name != "X":
        return oracle.run(circ)[0]
    ref = oracle.run(W.Circuit(circ.ops[:-1]))[0]
    i = np.arange(ref.size)
    on = np.all([(i >> c) & 1 for c in last.controls], axis=0)
    return ref[np.where(on, i ^ (1 << last.targets[0]), i)]


def _not_finite(n, kind, far):
    """RX of a NaN angle where qubit 1 is 1, then controlled gates on qubit 1,
    whose pairs have one member there, under the control of another qubit."""
    c = n - 1 if far else 2
    ops = [W.add_qubits(n), W.add_cbits(1)] + [W.gate("RY", [q], params=(0.5 + 0.05 * q,)) for q in range(n)]
    ops += [W.gate("RX", [0], controls=[1], params=(float("nan"),))]
    if kind == "cond":
        ops += [W.gate("H", [1], conds=[(0, 1)])]   # (cbit 0 is 0)
    elif kind == "X":
        ops += [W.gate("X", [1], controls=[c, 3])]
    else:
        ops += [W.gate(kind, [1], controls=[c], params=(0.8,) if kind in ("RX", "RY") else ())]
    return W.Circuit(ops, label=f"not_finite_{kind}_n{n}")


@pytest.mark.parametrize("kind", ["RX", "RY", "H", "Y", "X", "cond"])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_values_that_are_not_finite_stay_where_they_are(dtype, kind):
    """Pairs off a gate's controls keep their values: the amplitudes that are
    not finite are the oracle's, in one chunk, staged jobs and stages."""
    import paper_1908_07187_amd as qk
    b, circs, got = qk.Batch(dtype), [], []
    for n, far in ((5, False), (5, True), (9, True), (15, False), (15, True)):
        circs.append(_not_finite(n, kind, far))
        qk.add_circuit(b, circs[-1])
    b.run()
    b.sync()
    got += [b.state(j) for j in range(len(circs))]
    b.close()
    for far in (False, True):
        circs.append(_not_finite(14, kind, far))
        s = qk.Sim(dtype)
        s.set_tuning("stages", 1)
        qk.Program(circs[-1]).run(s)
        got.append(s.state())
        s.close()
    for c, g in zip(circs, got):
        ref = _reference(c)
        fine = np.isfinite(ref)
        print(f"[gpu-stage-limits] {c.label} {dtype}: {int(fine.sum())} finite of {fine.size}", flush=True)
        assert 0 < fine.sum() < fine.size
        assert np.array_equal(np.isfinite(g), fine)
        assert np.max(np.abs(g.astype(np.complex128) - ref)[fine]) <= (1e-12 if dtype == "c128" else 1e-5)
