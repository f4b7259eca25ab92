"""Reading and setting a run's state does not depend on the calling thread's
current device: the library on a host that plays two devices (no GPU)."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2404_01159_amd", "librvea.so")

SCRIPT = """
import ctypes as C, sys
shim, lib = C.CDLL(sys.argv[1]), C.CDLL(sys.argv[2])
at, home, stream = int(sys.argv[3]), int(sys.argv[4]), C.c_void_p(int(sys.argv[5], 0))
K, d, m = 6, 4, 3
need = C.c_size_t(0)
args = (1, m, d, C.c_int64(K), C.c_int64(K))
assert lib.rvea_footprint(*args, None, C.byref(need)) == 0
ws = C.create_string_buffer(need.value + 256)
base = C.c_void_p((C.addressof(ws) + 255) // 256 * 256)
run = C.c_void_p(0)
shim.two_devices(at, home)
st = lib.rvea_create(*args, C.c_uint64(1), None, base, need, stream, C.byref(run))
assert st == 0, ("create", st)
X, F, V, g = (C.c_float * (K * d))(), (C.c_float * (K * m))(), (C.c_double * (K * m))(), (C.c_double * K)()
valid, t = (C.c_uint8 * K)(), C.c_int64(0)
V[0:K * m] = [1.0] * (K * m)
for cur in (0, 1):
    shim.two_devices(cur, home)
    st = lib.rvea_get_state(run, X, F, valid, V, None, g, C.byref(t))
    assert st == 0, ("get", cur, st)
    for gamma in (None, g):
        st = lib.rvea_set_state(run, X, F, valid, V, gamma, C.c_int64(3))
        assert st == 0, ("set", cur, st)
    assert shim.two_devices_current() == cur
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    cc = shutil.which("gcc")
    if cc is None:
        pytest.skip("no gcc")
    out = str(tmp_path_factory.mktemp("devices") / "two_devices.so")
    subprocess.run([cc, "-shared", "-fPIC", "-O1", "-w", os.path.join(HERE, "golden", "two_devices.c"),
                    "-o", out], check=True)
    return out


# the current device at creation, the run's device, its stream
@pytest.mark.parametrize("at,home,stream", [(0, 0, "0"), (1, 1, "0"), (0, 0, "0x100"), (1, 1, "0x101"),
                                            (0, 1, "0x101")])
def test_state_of_a_run_on_another_device(shim, at, home, stream):
    preload = " ".join(x for x in (shim, os.environ.get("LD_PRELOAD")) if x)
    r = subprocess.run([sys.executable, "-c", SCRIPT, shim, LIB, str(at), str(home), stream],
                       env=dict(os.environ, LD_PRELOAD=preload), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
