"""Host memory that runs out comes back as an error code (no GPU)."""
import os
import subprocess
import sys

import pytest

pytest.importorskip("paper_2509_21037_amd")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# plan creation under more and more address space, until the host tables fit
CHILD = r"""
import ctypes, resource, sys
import scgen
from paper_2509_21037_amd import scasm
lib = scasm.load()
subs = [scgen.box_subdomain("heat", (90, 90), 1.0 / 90, 3)] * 24
keep = []
descs = (scasm.SubdomainDesc * len(subs))()
for d, s in zip(descs, subs):
    scasm._fill_desc(d, s, keep)
opt = scasm._options(n_threads=1)
vm = [int(l.split()[1]) for l in open("/proc/self/status") if l.startswith("VmSize")][0] * 1024
codes = []
for kb in range(0, 400000, 250):
    h = ctypes.c_void_p()
    resource.setrlimit(resource.RLIMIT_AS, (vm + kb * 1024, -1))
    codes.append(lib.sc_plan_create(descs, len(subs), ctypes.byref(opt), None, ctypes.byref(h)))
    resource.setrlimit(resource.RLIMIT_AS, (-1, -1))
    assert not h.value
    if codes[-1] != scasm.SC_ERR_OOM:
        break
print(codes.count(scasm.SC_ERR_OOM), codes[-1])
"""


def test_plan_creation_out_of_memory():
    """SC_ERR_OOM at every point where an allocation of the planner or of the
    plan's tables fails, then (without a device) SC_ERR_DEVICE: no exception
    leaves the call, the process lives on."""
    env = dict(os.environ, OMP_NUM_THREADS="1", HIP_VISIBLE_DEVICES="", PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", CHILD], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, env=env,
                       cwd=ROOT, timeout=300)
    assert r.returncode == 0, r.stderr[-500:]
    oom, last = r.stdout.split()[-2:]
    assert int(oom) > 3 and int(last) == 4
