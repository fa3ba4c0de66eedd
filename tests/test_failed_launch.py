"""What a call whose launch fails half way leaves to the next one, on the host alone: libef.so over a runtime that lists the kernels
instead of running them (fake_hip.c)."""
import os
import subprocess
import sys

import paper_1905_10936_amd as ef

HERE = os.path.dirname(os.path.abspath(__file__))

DRIVER = r"""
import ctypes, sys
fake, L = ctypes.CDLL(sys.argv[1]), ctypes.CDLL(sys.argv[2])
fake.fake_launched.restype = ctypes.c_char_p
vp, i64, f32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_float
d, n = 3 * 4096 * 9 + 77, 2
offs = (i64 * 4)(0, 4096 * 5 + 3, 4096 * 9, d)
plan = vp()
assert L.ef_plan_create(ctypes.byref(plan), offs, i64(3), n, None) == 0
ds = (d + 3) // 4 * 4
keep = []
def buf(size):
    b = (ctypes.c_char * (size + 64))()
    keep.append(b)
    return vp((ctypes.addressof(b) + 63) // 64 * 64)
v, m, e, words, scales, out = buf(4 * n * ds), buf(4 * n * ds), buf(4 * n * ds), buf(8 * n * ds), buf(4 * n * 3), buf(16 * n)
calls = {
    "own": lambda: L.ef_compressor_quality(plan, n, v, i64(ds), out, None),
    "static": lambda: L.ef_compressor_quality_static(plan, n, v, i64(ds), out, None),
    "worker": lambda: L.ef_worker_step_quality(plan, n, v, i64(ds), m, e, i64(ds), f32(.9), f32(.1), f32(.1), words, scales, out, None),
}
def run(name, fail):
    fake.fake_begin(fail)
    rc = calls[name]()
    return rc, [k for k in fake.fake_launched().decode().split() if "quality" in k or "worker" in k]
def is_reset(names):
    return ["k_quality_reset" in k for k in names]
for first in calls:
    rc, whole = run(first, -1)
    assert rc == 0 and len(whole) == 2 and not any(is_reset(whole)), whole
    assert "k_quality_blocks" in whole[-1]
    for second in calls:
        rc, names = run(first, 1)               # the second of the two
        assert rc != 0 and names == whole[:1], (first, names)
        rc, names = run(second, -1)
        assert rc == 0 and is_reset(names) == [True, False, False], (first, second, names)
        rc, names = run(second, -1)
        assert rc == 0 and is_reset(names) == [False, False], names
print("failed launches ok")
"""


def test_diagnostics_after_a_launch_that_failed(tmp_path):
    ef.lib()
    fake = str(tmp_path / "fake_hip.so")
    subprocess.run([os.environ.get("CC", "gcc"), "-O1", "-shared", "-fPIC", "-w", "-o", fake, os.path.join(HERE, "fake_hip.c")], check=True)
    run = subprocess.run([sys.executable, "-c", DRIVER, fake, ef.LIB_PATH], capture_output=True, text=True, timeout=120,
                         env=dict(os.environ, LD_PRELOAD=fake))
    assert run.returncode == 0, run.stdout + run.stderr
    assert "failed launches ok" in run.stdout
