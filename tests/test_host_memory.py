"""gs_init_gap where host memory is short: an error, never an exception through the C entry,
and one copy of the beam schedules, not several.  (No device is needed: the copies come
before the first device call.)"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes as C, resource, sys
import numpy as np
from paper_2603_24010_amd import gapsim, workloads as W
n, room = 1 << 26, int(sys.argv[1])
lib = gapsim.lib()
arr = (gapsim.GsGapParams * 1)()
cfg = W.config_tesla().replace(beam_schedule=np.zeros(n, dtype=np.int64))
arr[0] = gapsim.params_from(cfg, 32, (10, 10))
h = C.c_void_p()
alloc = gapsim.GsAllocator(gapsim.ALLOC_FN(lambda nbytes, user: None), gapsim.RELEASE_FN(lambda p, user: None), None)
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + room, used + room))
rc = lib.gs_init_gap(C.byref(h), 1, arr, C.byref(alloc), None)
print("status", rc, bool(h.value), lib.gs_last_error(None).decode())
"""


@pytest.mark.parametrize("room_mib,says", [
    (128, "out of host memory"),  # the copy of the schedule (512 MiB) does not fit
    (768, "allocation of"),       # it fits, once; the device (or its pinned memory) is what is missing
])
def test_short_host_memory_is_an_error(room_mib, says):
    r = subprocess.run([sys.executable, "-c", CHILD, str(room_mib << 20)], capture_output=True, text=True, cwd=ROOT,
                       timeout=100)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    status, made, msg = r.stdout.split("status ")[1].split(" ", 2)
    assert (int(status), made) == (-2, "False") and says in msg, r.stdout
