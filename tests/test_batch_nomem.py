"""A batched plan whose host tables do not fit in memory: dvr_batch_create returns DVR_E_NOMEM, and no exception
leaves the C entry (on the CPU, in a process with a bounded address space; the view array is never reached)."""
import subprocess
import sys
from pathlib import Path


ROOT = Path(__file__).resolve().parents[1]
CHILD = r"""
import ctypes as C, resource, sys
from paper_2605_19737_amd import _abi as abi
L = abi.load()
FAKE = 0x10000
vm = [int(l.split()[1]) for l in open("/proc/self/status") if l.startswith("VmSize")][0] * 1024
vols = (abi.BatchVolume * 1)()
vols[0] = abi.BatchVolume(FAKE, abi.DVR_F32, abi.Grid(8, 9, 10, 1.0, 1.0, 1.0),
                          abi.FeaturesBuf(FAKE, FAKE, FAKE, FAKE, abi.DVR_F32, abi.DVR_PLANAR, None, None))
d = abi.BatchDesc()
d.nvol, d.vols = 1, vols
d.nview, d.views = 20000000, C.cast(FAKE, C.POINTER(abi.BatchView))
d.fp.nsigma = 1
d.fp.sigma_mm[0] = 1.0
d.fp.alpha = d.fp.beta = 0.5
d.fp.c, d.fp.eig_gap_fp64 = 0.2, 1e-3
plan = C.c_void_p()
resource.setrlimit(resource.RLIMIT_AS, (vm + (1 << 29), resource.RLIM_INFINITY))
s = L.dvr_batch_create(C.byref(d), C.byref(plan))
print("status", s, bool(plan.value), flush=True)
"""


def test_plan_without_host_memory():
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split() == ["status", "-5", "False"]
