"""Stages and fused blocks on one simulator, as the autotuner sets them: gates
that the stage queue does not take (user matrices, five controls, more than two
conditions), with few or many builtins between them, short queues, captured
gates and states below one chunk.  Against the oracle.

Tolerance: a gate costs at most 6 u over the 2-norm by itself (two roundings and
a rounded coefficient per product) and not more as part of a composed block of
up to 5 qubits, whose rows hold at most 32 complex products: 64 u per block, over
at most every second gate."""
import numpy as np
import pytest

import oracle
import workloads as W
from workloads.circuits import rng_for

pytestmark = pytest.mark.gpu


def _sim(dtype, n):
    import paper_1908_07187_amd as qk
    s = qk.Sim(dtype)
    s.set_tuning("stages", 1)
    s.set_fusion(5 if n >= 13 else 3)
    return s


def _check(circ, dtype, got, ref=None):
    ref = oracle.run(circ)[0] if ref is None else ref
    d = float(np.max(np.abs(got.astype(np.complex128) - ref)))
    tol = 32 * len(circ.gate_ops()) * (2.0 ** -53 if dtype == "c128" else 2.0 ** -24) + 1e-13
    print(f"[gpu-stage-fusion] {circ.label} {dtype}: max|d| = {d:.2e} (tol {tol:.2e})", flush=True)
    assert d <= tol


def _mixed(n, gaps, seed):
    """Runs of builtins of the given lengths, and between them in turn a user
    matrix on 1 to 3 qubits, one with a control, five controls, three
    conditions, a measurement and a SWAP (relabelled)."""
    rng = rng_for(seed)
    ops, user = [W.add_qubits(n), W.add_cbits(3)] + [W.gate("RY", [q], params=(0.4 + 0.1 * q,)) for q in range(n)], {}
    one = ["H", "X", "T", "RX", "RY", "RZ"]
    for k, gap in enumerate(gaps):
        for _ in range(gap):
            q = [int(x) for x in rng.permutation(n)[:3]]
            r = int(rng.integers(9))
            if r < 6:
                ops.append(W.gate(one[r], q[:1], params=(float(rng.uniform(0, 6)),) if r >= 3 else ()))
            else:
                ops.append((W.gate("X", q[:1], controls=q[1:2 + r % 2]), W.gate("RZZ", q[:2], params=(0.7,)),
                            W.gate("CPHASE", q[:2], params=(1.1,)))[r - 6])
        q = [int(x) for x in rng.permutation(n)[:6]]
        m = k % 7
        if m < 3:
            user[f"U{k}"] = {"kind": "matrix", "k": m + 1, "matrix": W.random_unitary(m + 1, rng)}
            ops.append(W.gate(f"U{k}", q[:m + 1]))
        elif m == 3:
            user[f"U{k}"] = {"kind": "matrix", "k": 1, "matrix": W.random_unitary(1, rng)}
            ops.append(W.gate(f"U{k}", q[:1], controls=q[1:2]))
        elif m == 4:
            ops.append(W.gate("RX", q[:1], controls=q[1:], params=(0.9,)))
        elif m == 5:
            ops += [W.measure(q[0], cbit=0, u=0.37), W.gate("RY", q[1:2], conds=[(0, 0), (1, 0), (2, 0)], params=(0.8,))]
        else:
            ops += [W.gate("SWAP", q[:2]), W.gate("H", q[:1], conds=[(0, 1)])]
    return W.Circuit(ops, user_gates=user, label=f"mixed_n{n}_{'_'.join(map(str, gaps[:4]))}")


@pytest.mark.parametrize("dtype,n", [("c128", 12), ("c64", 13), ("c128", 15), ("c64", 16), ("c64", 24)])
@pytest.mark.parametrize("gaps", [[0] * 7, [1, 2] * 7, [3, 4, 5] * 5, [7, 8, 9] * 5, [20, 1, 0, 30, 2, 3, 5] * 2])
def test_gates_of_both_kinds_in_turn(dtype, n, gaps):
    import paper_1908_07187_amd as qk
    c = _mixed(n, gaps, 10 * n + len(gaps))
    ref, cb, recs = oracle.run(c)
    assert all(abs(r.u - r.P0) > 1e-6 for r in recs)
    s = _sim(dtype, n)
    qk.Program(c).run(s)
    got, bits = s.state(), list(s.read_cbits())
    s.close()
    assert bits == list(cb)
    _check(c, dtype, got, ref)


@pytest.mark.parametrize("dtype,n", [("c128", 5), ("c64", 9), ("c64", 12), ("c128", 14), ("c64", 14)])
def test_short_queues(dtype, n):
    """A flush after every one, two, three gates."""
    import paper_1908_07187_amd as qk
    from paper_1908_07187_amd.batch import op_array
    c = W.c2_random_rzz(n=n, depth=3, seed=n)
    s = _sim(dtype, n)
    s.add_qubits(n)
    gates = c.gate_ops()
    k = i = 0
    while i < len(gates):
        s.apply_ops(*op_array(W.Circuit(gates[i:i + 1 + k % 3])))
        s.flush()
        i += 1 + k % 3
        k += 1
    _check(c, dtype, s.state())
    s.close()


@pytest.mark.parametrize("dtype,n", [("c128", 14), ("c64", 14)])
def test_captured_gates_are_fused(dtype, n):
    """Capture holds nothing back for stages: the gates go by fused blocks, and
    every replay, with other work between, gives the state again."""
    import torch
    import paper_1908_07187_amd as qk
    c = W.c2_random_rzz(n=n, depth=4, seed=5)
    body = W.Circuit(c.gate_ops())
    s = qk.Sim(dtype, stream=torch.cuda.Stream())
    s.set_tuning("stages", 1)
    s.set_fusion(5)
    s.add_qubits(n)
    prog = qk.Program(body)
    ids = prog.define_gates(s)
    s.sync()
    s.capture_begin()
    s.reset()
    prog.run(s, ids=ids)
    g = s.capture_end()
    assert 2 * s.stats()["fused_blocks"] < len(body.ops)
    ref = oracle.run(c)[0]
    for _ in range(3):
        g.launch()
        _check(c, dtype, s.state(), ref)
        torch.zeros(1 << 20, device="cuda").add_(1).sum().item()
    g.close() if hasattr(g, "close") else None
    s.close()


@pytest.mark.parametrize("dtype,n", [("c128", 10), ("c128", 11), ("c64", 11), ("c64", 12)])
def test_stretches_of_diagonal_gates_below_one_chunk(dtype, n):
    """A QFT (few passes for many gates: passes of their own), also around a
    user matrix, and the blocks of a circuit that has no such stretches."""
    import paper_1908_07187_amd as qk
    from workloads.circuits import big_endian_bits
    head = [W.add_qubits(n)] + [W.gate("RY", [q], params=(0.3 + 0.2 * q,)) for q in range(n)]
    qft = W.qft_ops(big_endian_bits(n))
    user = {"U": {"kind": "matrix", "k": 2, "matrix": W.random_unitary(2, rng_for(n))}}
    circs = [W.Circuit(head + qft + [W.gate("U", [1, n - 1])] + qft, user_gates=user, label=f"qft_n{n}"),
             W.c2_random_rzz(n=n, depth=2, seed=n)]
    blocks = []
    for c in circs:
        s = _sim(dtype, n)
        qk.Program(c).run(s)
        _check(c, dtype, s.state())
        blocks.append(s.stats()["sweeps"])
        s.close()
    assert blocks[0] < len(circs[0].gate_ops()) // 2 and blocks[1] < len(circs[1].gate_ops()) // 2
