"""What the entry points launch, seen from the host: the HIP runtime's place is taken by
tests/hip_recorder.c in a process of its own, so nothing runs and no GPU is needed."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, os, sys
import numpy as np
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
for f in ("lanes", "groups", "lds"):
    getattr(rec, "recorder_" + f).restype = ctypes.c_uint64
rec.recorder_kernel.restype = ctypes.c_char_p
sys.path.insert(0, os.getcwd())
import paper_2607_01203_amd as leb
L = leb.lib()
P = ctypes.c_void_p(1 << 40)                       # an aligned address; nothing reads it
def ok(rc):
    assert rc == 0, rc
def mlp(widths, nx):
    return leb.MLP([np.ones((b, a), np.float32) for a, b in zip(widths[:-1], widths[1:])],
                   [np.zeros(b, np.float32) for b in widths[1:]], nx, False)
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("recorder") / "hip_recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(ROOT, "tests", "hip_recorder.c"), "-ldl"],
                   check=True)
    return so


def _run(recorder, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, recorder], cwd=ROOT, capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_dynamic_lds_limit_on_every_device(recorder):
    """The limit of dynamic LDS is an attribute of the device: a kernel that uses more than
    64 KB finds it raised on whichever device is current, not only on the first one."""
    _run(recorder, """
dyn = leb.chain_dynamics(1)
net = mlp([16, 64, 64, 12], 12)
e = (ctypes.c_double * 6)(*[0.01] * 6)
opt = leb.FPOptions(1e-6, 2, 0.0, 1e-12, 0, 1e-6)
n = ctypes.c_int32()
big = 0
for d in (0, 1, 0, 2):
    rec.recorder_device(d)
    rec.recorder_clear()
    ok(L.leb_nn_bound(net.handle, 1, 1024, P, P, None, P, None, P, P, None, None, 0.0, None, None))
    ok(L.leb_nn_backward(net.handle, 1, 1024, P, P, None, P, P, P, P, P, None, P, None))
    ok(L.leb_tube_map(1, 83, 1, P, e, P, P, P, P, None))
    ok(L.leb_fixed_point_solve_noalloc(ctypes.byref(dyn), 1, 200, P, P, P, e, ctypes.byref(opt), P, P, P,
                                       ctypes.byref(n), None))
    ok(L.leb_sls_fixed_point(ctypes.byref(dyn), 1, 300, P, P, P, 0, None, 0.0, 0.0, P, P, P, P, P, None))
    big += sum(rec.recorder_lds(i) > 65536 for i in range(rec.recorder_launches()))
    assert rec.recorder_refused() == 0, (d, rec.recorder_refused())
assert big >= 4 * 5, big
""")


def test_small_systems_lanes_per_row(recorder):
    """A row of a small system takes about as many lanes as it has Hessian entries (9, 3, 3
    and 1 of the 3-D quadrotor, the satellite and the two sine systems), whatever the form:
    lanes without an entry are what a large batch would wait for."""
    _run(recorder, """
J3 = (1.0, 2.0, 3.0)
for dyn, G in ((leb.quad3d_dynamics(0.05, 1.0, 9.81, J3), 16), (leb.satellite_dynamics(0.1), 4),
               (leb.sincos_dynamics(2), 4), (leb.sincos_dynamics(1), 1)):
    for mode in (0, 1, 2):
        for units in (1, 1000, 1000003):
            rec.recorder_clear()
            ok(L.leb_interval_hessian_bound(ctypes.byref(dyn), mode, 1, units, P, P, P, P, P, P, P, None))
            assert rec.recorder_launches() == 1
            lanes = rec.recorder_lanes(0)
            assert units * dyn.nx <= lanes <= (units + 64 // G) * dyn.nx * G + 256, (dyn.kind, units, lanes)
""")


def test_causal_pass_workgroups_of_large_batches(recorder):
    """The one-launch causal pass of a batch that fills the chip more than once: workgroups
    of four waves while the horizon is short, so that three share a compute unit; the wide
    ones up to one a compute unit."""
    _run(recorder, """
for U in (2, 3, 4, 5):
    dyn = leb.chain_dynamics(U)
    for batch, narrow in ((1, False), (256, False), (257, True), (8192, True)):
        rec.recorder_clear()
        ok(L.leb_sls_fixed_point(ctypes.byref(dyn), batch, 8, P, P, P, 0, None, 0.0, 0.0, P, P, P, P, P, None))
        i = rec.recorder_launches() - 1
        assert b"sls_fp_chain" in rec.recorder_kernel(i)
        lanes = rec.recorder_lanes(i) // rec.recorder_groups(i)
        assert rec.recorder_groups(i) == batch and (lanes <= 256) == narrow, (U, batch, lanes)
""")


def test_descent_of_many_steps_in_many_launches(recorder):
    """The descent of few timesteps is one launch while that launch is short; a call of any
    number of steps does not hold the device in one."""
    _run(recorder, """
dyn = leb.chain_dynamics(2)
for steps, one in ((0, True), (10, True), (1000, True), (10 ** 4, False)):
    rec.recorder_clear()
    ok(L.leb_pgd_nominal(ctypes.byref(dyn), 1, 40, P, P, None, P, 0, 1.0, steps, 0.25, P, P, P, P, None))
    assert (rec.recorder_launches() == 1) == one, (steps, rec.recorder_launches())
""")
