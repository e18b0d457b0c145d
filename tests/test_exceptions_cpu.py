"""C++ exceptions stay inside: an entry of the C ABI returns a status where the host's memory runs out, and the compiled marshalling
takes an exception of the call it made neither for arguments that are not plain nor into the interpreter without its lock."""
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

# the marshalling's own call(), around a call that throws
THROWING = r"""
#include <new>
#include "arguments.cpp"
static int calls = 0;
static PyObject* throwing(PyObject*, PyObject* const* argv, Py_ssize_t n) {
    return call(argv, n, 0, [](Args&) { return []() -> int { ++calls; throw std::bad_alloc(); }; });
}
static PyObject* count(PyObject*, PyObject*) { return PyLong_FromLong(calls); }
static PyMethodDef table[] = {{"throwing", FAST(throwing)}, {"count", count, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef def = {PyModuleDef_HEAD_INIT, "throwing", nullptr, -1, table, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_throwing() { return PyModule_Create(&def); }
"""


def _run(code):
    return subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=110)


def test_host_memory_running_out_is_a_status():
    r = _run(NO_MEMORY.format(root=ROOT))
    assert r.returncode == 0 and "refused" in r.stdout, (r.returncode, r.stderr[-2000:])


def test_marshalling_survives_a_call_that_throws(tmp_path):
    from paper_2211_15023_amd import build
    src = tmp_path / "throwing.cpp"
    src.write_text(THROWING)
    os.symlink(build.SO, tmp_path / "libaccerl.so")
    build.compile_module(str(src), str(tmp_path / "throwing.so"), ["-I", build.CSRC])
    r = _run(f"import sys; sys.path[:0] = [{ROOT!r}, {str(tmp_path)!r}]\n"
             "import paper_2211_15023_amd as A; A.load_library()\n"
             "import throwing\n"
             "try: throwing.throwing()\n"
             "except RuntimeError as e: assert 'exception' in str(e)\n"
             "else: raise SystemExit('no error')\n"
             "assert throwing.count() == 1; print('said')")
    assert r.returncode == 0 and "said" in r.stdout, (r.returncode, r.stderr[-2000:])
