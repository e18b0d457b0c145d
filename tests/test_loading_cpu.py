"""What needs which file: host-only calls take libaccerl.so alone, the calls that go through accerl_args.so say how to build it where it is
missing or of another torch or Python."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import sys
sys.path[:0] = [{tmp!r}, {root!r}]
import numpy as np
import workloads as wl, paper_2211_15023_amd as A
assert A.__file__.startswith({tmp!r})
arch = A.make_arch(wl.CONFIGS[0]["teacher"], "fp32")
assert "steps=" in A.accerl_plan_describe(arch, np.zeros(A.blob_sizes(arch)[0], np.uint8))
assert A.accerl_mixture_alpha(0.5, 0.0, 1.0) == 0.5
for call, n in ((A.accerl_actor_forward, 6), (A.accerl_actor_forward_teacher, 6), (A.accerl_actor_forward_recurrent, 9),
                (A.accerl_monitor_kl, 5), (A.accerl_monitor_kl_noalloc, 5), (A.accerl_vtrace, 12)):
    try:
        call(*[None] * n)
    except ImportError as e:
        assert "accerl_args" in str(e) and "g.build()" in str(e), e
    else:
        raise SystemExit("no error")
print("said")
"""


@pytest.mark.parametrize("there", ["missing", "not loadable"])
def test_without_the_compiled_marshalling(tmp_path, there):
    import paper_2211_15023_amd as A
    pkg = tmp_path / "paper_2211_15023_amd"
    pkg.mkdir()
    here = os.path.dirname(A.__file__)
    for f in ("__init__.py", "binding.py"):
        shutil.copy(os.path.join(here, f), pkg)
    os.symlink(os.path.join(here, "libaccerl.so"), pkg / "libaccerl.so")
    if there != "missing":
        (pkg / "accerl_args.so").write_text("of another build")
    r = subprocess.run([sys.executable, "-c", CHILD.format(tmp=str(tmp_path), root=ROOT)], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and "said" in r.stdout, (r.returncode, r.stderr[-2000:])
