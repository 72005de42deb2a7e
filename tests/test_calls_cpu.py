"""The native marshalling of calls on the host: the interpreter's end inside a call, another torch, a machine that cannot build it."""
import os
import subprocess
import sys

import pytest

# the library's function replaced by one that only waits, the stream by none
PROBE = r"""
#include <c10/hip/HIPStream.h>
#include <unistd.h>
namespace c10::hip {
struct NoStream {
    void* stream() const { return nullptr; }
};
inline NoStream no_stream() { return {}; }
}
#define getCurrentHIPStream no_stream
#include "calls.cpp"
namespace {
PyObject* wait_call(PyObject*, PyObject* const*, Py_ssize_t n) {
    return guarded<0>(n, [] { return made("wait", [](hb_stream) { usleep(300000); return HB_OK; }); });
}
PyMethodDef probe_methods[] = {{"wait", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(wait_call)), METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef probe_module = {PyModuleDef_HEAD_INIT, "probe_calls", nullptr, -1, probe_methods, nullptr, nullptr, nullptr, nullptr};
}
PyMODINIT_FUNC PyInit_probe_calls() {
    PyObject* calls = PyInit__calls();
    if (!calls) return nullptr;
    Py_DECREF(calls);
    g_error = PyExc_RuntimeError;
    return PyModule_Create(&probe_module);
}
"""
PROGRAM = """
import threading
import torch, probe_calls
inside = threading.Event()
def calls():
    while True:
        inside.set()
        assert probe_calls.wait() is True
threading.Thread(target=calls, daemon=True).start()
inside.wait()
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    """Runs a program that can import the probe."""
    import __graft_entry__ as entry
    if entry._calls_wants():
        pytest.skip("cannot be built here: no " + ", ".join(entry._calls_wants()))
    d = tmp_path_factory.mktemp("calls")
    source = d / "probe_calls.cpp"
    source.write_text(PROBE)
    entry._build_calls(str(source), str(d / "probe_calls"))
    path = os.pathsep.join([str(d), os.path.dirname(os.path.dirname(os.path.abspath(__file__)))])
    return lambda program: subprocess.run([sys.executable, "-c", program], env={**os.environ, "PYTHONPATH": path}, capture_output=True, text=True, timeout=100)


def test_a_daemon_thread_in_a_call_does_not_abort_the_program_at_its_end(run):
    r = run(PROGRAM)
    assert r.returncode == 0, r.stderr


@pytest.mark.parametrize("other", ["2.10.0", "+other", ".post1"])       # the same release from somewhere else, too
def test_another_torch_does_not_load_it(run, other):
    r = run(f"""
import torch
v = torch.version.__version__
torch.version.__version__ = {other!r} if {other!r}[0] == "2" else v + {other!r}
try:
    import probe_calls
except ImportError as e:
    assert "built with torch " + v in str(e), e
else:
    raise SystemExit("loaded")
""")
    assert r.returncode == 0, r.stdout + r.stderr


def test_a_library_without_it_says_so_and_works():
    program = """
import sys
sys.modules["paper_2512_02371_amd._calls"] = None                       # an import of it fails
from paper_2512_02371_amd import hb
hb.load()
assert hb._calls is None and hb.hb_sat2d_workspace_size(64, 64) > 0
"""
    r = subprocess.run([sys.executable, "-c", program], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "native marshalling" in r.stderr, r.stderr


def test_it_is_not_asked_for_where_it_cannot_be_built(monkeypatch):
    import shutil
    import __graft_entry__ as entry
    which = shutil.which
    monkeypatch.setattr(shutil, "which", lambda name, *a, **k: None if name == "g++" else which(name, *a, **k))
    assert "g++" in entry._calls_wants()
