"""LDS circuits with gates past 45 degrees, which run as quarter turns kept by the
host (bit flips and Z of the frame, factors i of the state) and what is left:
every kind of gate behind them, across stages and measurements, with nothing or
only flips behind the last one; and the error of complex64 stages against fused
blocks.

Tolerance: a gate changes an amplitude by at most 4 u of the state's norm (u =
2^-53 or 2^-24), a pass by 2 u more: 6 u per gate, plus 1e-13 for the oracle's own
rounding."""
import numpy as np
import pytest

import oracle
import workloads as W
from workloads.circuits import big_endian_bits, rng_for

pytestmark = pytest.mark.gpu


def _turns(n, seed, tail):
    """Far rotations of every kind (odd numbers of each, so that factors i stay),
    then in turn every gate that a Z or a flip of the frame meets."""
    rng = rng_for(seed)
    ops = [W.add_qubits(n), W.add_cbits(2)] + [W.gate("RY", [q], params=(0.3 + 0.17 * q,)) for q in range(n)]

    def far():
        return float(rng.choice([-1, 1]) * rng.uniform(np.pi / 2, np.pi) + rng.choice([0, 2 * np.pi]))

    for k in range(14):
        a, b, c, d = [int(x) for x in (list(rng.permutation(n)) * 4)[:4]]
        two, three = n > 1, n > 2
        ops += [W.gate("RX", [a], params=(far(),)), W.gate("RZ", [b], params=(far(),)), W.gate("RY", [c], params=(far(),))]
        if two:
            ops += [W.gate("RZZ", [a, b], params=(far(),)), W.gate("X", [a], controls=[b])]
        kind = k % 14
        if kind < 4 and two:
            ops.append(W.gate(("H", "RY", "RX", "Y")[kind], [b], controls=[a], params=(far(),) if kind in (1, 2) else ()))
        elif kind < 6 and three:
            ops.append(W.gate("X", [a], controls=[b, c][:kind - 3] + ([d] if n > 3 else [])))
        elif kind == 6 and two:
            ops.append(W.gate("SWAP", [a, b], controls=[c] if three else []))
        elif kind == 7 and two:
            ops.append(W.gate("CPHASE", [a, b], params=(0.4,)))
        elif kind == 8:
            ops += [W.measure(a, cbit=0, u=0.41), W.gate("RX", [a], conds=[(0, 1)], params=(far(),))]
        elif kind == 9:
            ops += [W.gate("X", [a]), W.gate("Y", [b]), W.gate("H", [a]), W.gate("Z", [c])]
        elif kind == 10 and two:
            ops.append(W.gate("RZ", [a], controls=[b], params=(far(),)))
        elif kind == 11 and two:
            ops.append(W.gate("PHASE", [a], controls=[b], params=(2.9,)))
        else:
            ops.append(W.gate("T", [a]))
    ops += {"none": [], "flips": [W.gate("X", [0]), W.gate("X", [n - 1], controls=[0] if n > 1 else [])],
            "measure": [W.measure(n - 1, cbit=1, u=0.63)], "turn": [W.gate("RZ", [n // 2], params=(far(),))]}[tail]
    return W.Circuit(ops, label=f"turns_n{n}_{tail}")


def _check(circ, got, dtype):
    ref, _, recs = oracle.run(circ)
    assert all(abs(r.u - r.P0) > 1e-6 for r in recs)
    d = float(np.max(np.abs(got.astype(np.complex128) - ref)))
    tol = 6 * len(circ.gate_ops()) * (2.0 ** -53 if dtype == "c128" else 2.0 ** -24) + 1e-13
    print(f"[gpu-turns] {circ.label} {dtype}: max|d| = {d:.2e} (tol {tol:.2e})", flush=True)
    assert d <= tol


@pytest.mark.parametrize("tail", ["none", "flips", "measure", "turn"])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_batch_jobs(dtype, tail):
    import paper_1908_07187_amd as qk
    top = 13 if dtype == "c128" else 14
    circs = [_turns(n, 3 * n + len(tail), tail) for n in (1, 2, 3, 4, 5, 7, 10, top, top + 1, top + 4)]
    b = qk.Batch(dtype)
    ids = [qk.add_circuit(b, c) for c in circs]
    b.run()
    b.sync()
    for c, j in zip(circs, ids):
        assert list(b.cbits(j)) == list(oracle.run(c)[1])
        _check(c, b.state(j), dtype)
    b.close()


@pytest.mark.parametrize("tail", ["none", "flips", "turn"])
@pytest.mark.parametrize("dtype,n", [("c128", 12), ("c128", 17), ("c64", 13), ("c64", 18)])
def test_stages(dtype, n, tail):
    import paper_1908_07187_amd as qk
    c = _turns(n, n + len(tail), tail)
    s = qk.Sim(dtype)
    s.set_tuning("stages", 1)
    qk.Program(c).run(s)
    _check(c, s.state(), dtype)
    s.close()


@pytest.mark.parametrize("n", [14, 18, 20])
def test_complex64_stages_are_as_exact_as_fused_blocks(n):
    """A QFT and its inverse, phases between them: the stages' error over that of
    3- to 5-qubit blocks, whose matrices are composed in 64 bits, is at most 1
    (the largest of theirs)."""
    import paper_1908_07187_amd as qk
    th = rng_for(n).uniform(0.2, np.pi - 0.2, n)
    qft, back = (W.qft_ops(big_endian_bits(n), inverse=inverse) for inverse in (False, True))
    c = W.Circuit([W.add_qubits(n)] + [W.gate("RY", [q], params=(float(th[q]),)) for q in range(n)] + qft
                  + [W.gate("RZ", [q], params=(float(th[q]),)) for q in range(n)] + back, label=f"qft_n{n}")
    ref = oracle.run(c)[0]
    err = {}
    for k in (0, 3, 4, 5):
        s = qk.Sim("c64")
        s.set_fusion(k)
        s.set_tuning("stages", k == 0)
        qk.Program(c).run(s)
        err[k] = float(np.linalg.norm(s.state().astype(np.complex128) - ref))
        s.close()
    print(f"[gpu-turns] {c.label}: {err}", flush=True)
    assert err[0] <= max(err[3], err[4], err[5])
