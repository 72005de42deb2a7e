"""The native marshalling of calls when the interpreter ends while a daemon thread is inside a call."""
import os
import subprocess
import sys

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


def test_a_daemon_thread_in_a_call_does_not_abort_the_program_at_its_end(tmp_path):
    import __graft_entry__ as entry
    source = tmp_path / "probe_calls.cpp"
    source.write_text(PROBE)
    entry._build_calls(str(source), str(tmp_path / "probe_calls.so"))
    r = subprocess.run([sys.executable, "-c", PROGRAM], env={**os.environ, "PYTHONPATH": str(tmp_path)}, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr
