"""Deferred measurement where its orders change: shots at 1, 2, 63 to 65 and
more chunks of the cumulative sums (the 64-way search), and distributions whose
listed qubits lie within a 128-byte line, in any order of the list.

The drawn index is compared with numpy's cumulative sum for every draw farther
than 1e-12 from an interval's end (both sums are in FP64, 2^21 positive terms:
rounding below 1e-12).  A distribution's entry is a sum of at most 2^14 / 256
terms per thread in order, a tree and 2^7 slabs: below 300 u = 4e-14 of it."""
import numpy as np
import pytest

import workloads as W
from workloads.circuits import rng_for

pytestmark = pytest.mark.gpu


def _sim(n, dtype, seed):
    import paper_1908_07187_amd as qk
    rng = rng_for(seed)
    ops = [W.add_qubits(n)] + [W.gate("RY", [q], params=(float(rng.uniform(0.4, 2.7)),)) for q in range(n)]
    ops += [W.gate("X", [(q + 1) % n], controls=[q]) for q in range(n)]
    s = qk.Sim(dtype)
    qk.Program(W.Circuit(ops)).run(s)
    p = np.abs(s.state().astype(np.complex128)) ** 2
    return s, p, rng


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [5, 14, 15, 16, 20, 21])
def test_shots(n, dtype):
    s, p, rng = _sim(n, dtype, n)
    u = np.concatenate([[0.0, 1.0 - 2.0 ** -53], rng.random(3000)])
    got = s.sample(u).astype(np.int64)
    s.close()
    c = np.cumsum(p)
    want = np.minimum(np.searchsorted(c, u * c[-1], side="right"), len(p) - 1)
    lo = np.where(want > 0, c[want - 1], 0.0)
    clear = (np.abs(u * c[-1] - lo) > 1e-12) & (np.abs(u * c[-1] - c[want]) > 1e-12)
    clear[0] = False
    assert clear.sum() > 2900
    print(f"[gpu-sampling] n={n} {dtype}: {int(clear.sum())} draws", flush=True)
    assert np.array_equal(got[clear], want[clear])
    assert p[got].min() > 0


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n,qubits", [(5, [0]), (9, [2, 0, 8]), (12, [11, 3, 1]), (16, [15, 0, 7, 2, 3, 1]),
                                      (21, [1, 20, 7, 15, 0]), (21, [4, 5]), (10, list(range(9, -1, -1)))])
def test_distributions(n, qubits, dtype):
    s, p, _ = _sim(n, dtype, 7 * n)
    got = s.probabilities(qubits)
    s.close()
    i = np.arange(1 << n)
    m = sum(((i >> q) & 1) << j for j, q in enumerate(qubits))
    want = np.bincount(m, weights=p, minlength=1 << len(qubits)) / p.sum()   # (a distribution is normalised)
    print(f"[gpu-sampling] n={n} {dtype} {qubits}: max|d| = {np.max(np.abs(got - want)):.1e}", flush=True)
    assert np.max(np.abs(got - want)) <= 1e-12
