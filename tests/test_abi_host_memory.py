"""Host memory that runs out inside the C ABI is an error code and a message, no
exception through the C frame.  In a process of its own whose address space is
limited once the library is loaded; no device work is reached."""
import os
import subprocess
import sys

import pytest

from paper_2108_02419_amd import _bbe

_CHILD = r"""
import ctypes, resource, sys
sys.path.insert(0, sys.argv[1])
import numpy as np
from paper_2108_02419_amd import _bbe
lib = _bbe.lib()
n = 8_000_000
kind, param = np.zeros(n, np.uint8), np.zeros(n, np.float32)
reqs = np.zeros(64, np.uint8)  # not looked at before the tables are there
out = ctypes.c_void_p(1)
kb = int([l for l in open("/proc/self/status") if l.startswith("VmSize")][0].split()[1])
soft, hard = resource.getrlimit(resource.RLIMIT_AS)
resource.setrlimit(resource.RLIMIT_AS, (kb * 1024 + (24 << 20), hard))
if sys.argv[2] == "plan":
    rc = lib.bbe_batch_plan_create(reqs.ctypes.data, n, 1, 1, None, None, 0, None,
                                   ctypes.byref(out))
else:
    rc = lib.bbe_bettors_create(kind.ctypes.data, param.ctypes.data, n, ctypes.byref(out))
resource.setrlimit(resource.RLIMIT_AS, (soft, hard))
print(rc, out.value, lib.bbe_last_error().decode())
"""


@pytest.mark.parametrize("what", ["plan", "bettors"])
def test_out_of_host_memory(what):
    if not os.path.exists(_bbe.LIB_PATH):
        pytest.skip("libbbe.so is not built")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    p = subprocess.run([sys.executable, "-c", _CHILD, root, what], capture_output=True, text=True,
                       timeout=240)
    assert p.returncode == 0, (p.returncode, p.stderr[-2000:])
    assert p.stdout.split(maxsplit=2)[:2] == [str(_bbe.ENOMEM), "None"], p.stdout
    assert "out of host memory" in p.stdout
