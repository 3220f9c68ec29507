"""Batch jobs on the host (no GPU): what qk_batch_add accepts, and the layout of
the gate loop that runs them."""
import ctypes as C
import math
import os
import re
import subprocess

import pytest

from paper_1908_07187_amd import qk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("n", [3, 20])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("value", [math.nan, math.inf, -math.inf, 1e308, 0.0])
def test_any_parameter_is_accepted(dtype, n, value):
    """Parameters are not checked, here as in the per-gate path: one that is
    not finite makes amplitudes that are not, and no error."""
    lib, h, job = qk.load(), C.c_void_p(), C.c_int32()
    assert lib.qk_batch_create(qk.DTYPES[dtype], None, None, C.byref(h)) == 0
    for name, targets in (("RX", 1), ("RY", 1), ("RZ", 1), ("PHASE", 1), ("CPHASE", 2), ("RZZ", 2)):
        for controls in (0, 1):
            o = qk.QkOp()
            o.kind, o.gate, o.n_targets, o.n_controls, o.param = qk.QK_OP_GATE, qk.BUILTINS[name], targets, controls, value
            o.targets[1], o.controls[0] = 1, 2
            assert lib.qk_batch_add(h, n, 0, C.byref(o), 1, C.byref(job)) == 0, (name, lib.qk_batch_last_error(h))
    assert lib.qk_batch_destroy(h) == 0


@pytest.mark.parametrize("width", ["f64", "f32"])
def test_every_place_of_the_gate_loop_goes_on_to_the_next_record(width):
    """Each place of the assembly gate loop moves the record pointer on, reads
    the next record, waits for it and works out the jump from it: one that did
    not would jump to itself for ever (read from the preprocessed source)."""
    src = open(os.path.join(ROOT, "paper_1908_07187_amd", "csrc", "batch.hip")).read()
    macros = src[src.index("#define QK_FETCH"):src.index("static_assert(kGateBytes == 512")]
    out = subprocess.run(["g++", "-E", "-P", "-x", "c++", "-"], input=macros + f"\nQK_GATE_LOOP({width})\n", text=True,
                         capture_output=True, check=True).stdout
    text = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', out[:out.rindex(": [a0]")])).replace("\\n", "\n").replace("\\t", "")
    places = re.split(r"LQKg(\d+)%=:\n", text)
    header = open(os.path.join(ROOT, "paper_1908_07187_amd", "csrc", "stage_records.h")).read()
    assert [int(k) for k in places[1::2]] == list(range(int(re.search(r"RG_OTHER = (\d+)", header).group(1))))
    for k, code in zip(places[1::2], places[2::2]):
        steps = ["s_add_u32 s84, s84, 48", "s_load_dwordx4 s[40:43], s[84:85]", "s_load_dwordx8 s[44:51], s[84:85]",
                 "s_waitcnt lgkmcnt(0)", "s_add_u32 s82, s80, s40", "s_setpc_b64 s[82:83]"]
        at = [code.find(s) for s in steps]
        assert -1 not in at and at == sorted(at), (k, at)


@pytest.fixture(scope="module")
def emulator(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("emulator") / "stage_records_emulator")
    csrc = os.path.join(ROOT, "paper_1908_07187_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                    "-I" + csrc, os.path.join(ROOT, "tests", "stage_records_emulator.cpp"), os.path.join(csrc, "stages.cpp"),
                    "-o", exe], check=True, capture_output=True, text=True)
    return exe


@pytest.mark.parametrize("seed", range(4))
def test_records_give_the_circuit(emulator, seed):
    """300 random circuits of up to 120 operations: the records, run as the
    interpreter runs them, against a plain simulation.  Both round each
    operation by at most 4 u of the norm (u = 2^-53), the records' scales by 2 u
    a pass: 120 (4 + 4 + 2) u = 1.4e-13."""
    r = subprocess.run([emulator, str(seed + 1), "300", "1.4e-13"], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
