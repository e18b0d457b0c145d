"""C++ exceptions stay inside: an entry of the C ABI returns a status where the host's memory runs out."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# 3136 -> 8192: 103 MB of weights, and 51 MB of constants that the plan has to build
NO_MEMORY = r"""
import resource, sys
sys.path.insert(0, {root!r})
import numpy as np
import workloads as wl, paper_2211_15023_amd as A
arch = A.make_arch(wl.nature_cnn("wide", fc=8192), "bf16")
blob = np.zeros(A.blob_sizes(arch)[0], np.uint8)
A.accerl_plan_describe(arch, blob)
used = [int(l.split()[1]) << 10 for l in open("/proc/self/status") if l.startswith("VmSize")][0]
resource.setrlimit(resource.RLIMIT_AS, (used + (16 << 20), used + (16 << 20)))
for i in range(2):
    try:
        A.accerl_plan_describe(arch, blob)
    except A.AccerlError as e:
        assert e.code == -2 and "host" in str(e), e
    else:
        raise SystemExit("planned without memory")
print("refused")
"""


def _run(code):
    return subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=110)


def test_host_memory_running_out_is_a_status():
    r = _run(NO_MEMORY.format(root=ROOT))
    assert r.returncode == 0 and "refused" in r.stdout, (r.returncode, r.stderr[-2000:])
