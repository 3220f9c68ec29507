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
