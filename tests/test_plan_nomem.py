"""Host memory that runs out while the launch plan is built (CPU only): a
status, as rc_cohort.h promises, and no C++ exception through the C entry."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# In a child process, which would abort: an address space limit just above
# what is in use, below the plan of four million one-session cohorts.
CHILD = """
import ctypes, resource
import numpy as np
from paper_2608_12123_amd import rc_cohort as rc
lib = rc.load_library()
off = np.arange((4 << 20) + 1, dtype=np.uint32)
table = np.zeros(16, dtype=np.uint32)
p32 = ctypes.POINTER(ctypes.c_uint32)
desc = rc.RcCohortDesc(off.size - 1, 4, 1, off.size - 1, off.ctypes.data_as(p32), table.ctypes.data_as(p32),
                       rc.RC_ROUTE_MOD, None, 32768)
n = ctypes.c_uint32(7)
with open("/proc/self/statm") as f:
    used = int(f.read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (20 << 20), resource.RLIM_INFINITY))
status = lib.rc_plan_lanes(ctypes.byref(desc), 256, None, None, 0, ctypes.byref(n))
resource.setrlimit(resource.RLIMIT_AS, (resource.RLIM_INFINITY, resource.RLIM_INFINITY))
assert status == rc.RC_E_NOMEM, status
assert n.value == 7
assert lib.rc_plan_lanes(ctypes.byref(desc), 256, None, None, 0, ctypes.byref(n)) == rc.RC_OK
assert n.value >= off.size - 1
"""


def test_plan_without_memory():
    res = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, (res.returncode, res.stdout + res.stderr)
