"""How a batch's cbits reach the host: read in every order of runs, refills and
ways of reading, and with memory for them first needed while another stream
captures."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _circuit(ones, zeros, n=6):
    """`ones` cbits that are 1, then `zeros` that are 0, of basis states."""
    ops = [W.add_qubits(n), W.add_cbits(ones + zeros), W.gate("X", [0])]
    ops += [W.measure(0, cbit=c, u=0.5) for c in range(ones)]
    ops += [W.measure(1, cbit=ones + c, u=0.5) for c in range(zeros)]
    return W.Circuit(ops)


def _fill(b, jobs):
    import paper_1908_07187_amd as qk
    b.clear()
    return [qk.add_circuit(b, _circuit(*j)) for j in jobs]


def _expect(jobs):
    return [[1] * j[0] + [0] * j[1] for j in jobs]


def test_cbits_of_every_refill():
    """More and fewer cbits each time, past one block of pinned memory, read by
    either call, both, or not at all."""
    import torch
    import paper_1908_07187_amd as qk
    b = qk.Batch("c128")
    for k, count in enumerate((1, 3, 40, 2, 300, 700, 5, 1200, 0, 30)):
        jobs = [((7 * j + k) % 129, (5 * j) % 120, 6 if j % 50 else 15) for j in range(count)] or [(0, 0)]
        ids, want = _fill(b, jobs), _expect(jobs)
        print(f"[gpu-cbits] refill {k}: {count} jobs, {b.sizes()[1]} cbits", flush=True)
        for _ in range(2):
            b.run()
            if k % 3 != 1:
                assert [list(b.cbits(j)) for j in ids] == want
            if k % 3 != 0:
                sb, cb = b.sizes()
                hs = torch.empty(sb, dtype=torch.uint8, pin_memory=True)
                hc = torch.empty(max(cb, 1), dtype=torch.uint8, pin_memory=True)
                b.read_async(hs.data_ptr(), sb, hc.data_ptr(), cb)
                b.sync()
                assert hc[:cb].tolist() == [x for j in want for x in j]
    b.close()


def test_cbits_read_after_asynchronous_reads_only():
    """A batch read by copies alone, then by qk_batch_read_cbits, before and
    after the next refill; and a second batch that takes its memory over."""
    import torch
    import paper_1908_07187_amd as qk
    b = qk.Batch("c64")
    hs, hc = torch.empty(1 << 16, dtype=torch.uint8, pin_memory=True), torch.empty(1 << 10, dtype=torch.uint8, pin_memory=True)
    for jobs in ([(3, 2), (0, 4)], [(4, 1)], [(1, 6), (7, 0)]):
        ids = _fill(b, jobs)
        b.run()
        b.read_async(hs.data_ptr(), hs.numel(), hc.data_ptr(), hc.numel())
        b.sync()
    assert [list(b.cbits(j)) for j in ids] == _expect(jobs)
    ids = _fill(b, [(2, 2)])
    b.run()
    assert [list(b.cbits(j)) for j in ids] == _expect([(2, 2)])
    b.close()
    b = qk.Batch("c64")
    ids = _fill(b, [(0, 5)])
    b.run()
    assert [list(b.cbits(j)) for j in ids] == _expect([(0, 5)])
    b.close()


def test_a_capture_on_another_stream_goes_on():
    """A batch whose cbits first need memory, and one that goes, while a stream
    of the same process captures (in the mode that forbids allocations)."""
    import torch
    import paper_1908_07187_amd as qk
    b, old = (qk.Batch("c128", stream=torch.cuda.Stream()) for _ in range(2))
    for x in (b, old):
        _fill(x, [(1, 0)])
        x.run()
        x.sync()
    jobs = [(60, 40)] * 1000
    ids = _fill(b, jobs)
    x, s, g = torch.zeros(1000, device="cuda"), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        g.capture_begin(capture_error_mode="global")
        x.add_(1)
        b.run()
        x.add_(1)
        g.capture_end()
    for k in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert x.eq(2 * (k + 1)).all()
    assert [list(b.cbits(j)) for j in (ids[0], ids[500], ids[-1])] == _expect(jobs[:3])
    b.close()
    old.close()
