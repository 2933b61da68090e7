"""A daemon thread that is inside a native call while the interpreter shuts down ends quietly, as in a ctypes call."""
import os
import subprocess
import sys

import pytest

from paper_2510_06175_amd import build

PROBE = r"""
#include "%s"
#include <unistd.h>
PyObject *nap(PyObject *, PyObject *const *, Py_ssize_t)
{
    return guarded([] { return without_gil([] { usleep(300000); return 0; }); });
}
PyMethodDef probe_methods[] = {VECINFER_METHOD(nap), {nullptr, nullptr, 0, nullptr}};
PyModuleDef probe_module = {PyModuleDef_HEAD_INIT, "_probe", nullptr, -1, probe_methods, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit__probe() { return PyModule_Create(&probe_module); }
"""

PROGRAM = r"""
import sys, threading, time
import torch
sys.path.insert(0, sys.argv[1])
import _probe
assert _probe.nap() == 0

class Linger:                       # keeps the shutdown, once begun, waiting for the thread's call to end
    def __del__(self, sleep=time.sleep):
        sleep(1)

linger = Linger()
threading.Thread(target=_probe.nap, daemon=True).start()
print("leaving", flush=True)
"""


def test_daemon_thread_at_shutdown(tmp_path):
    command = build.fastcall_command()
    if command is None:
        pytest.skip("no Python headers: the native module is not built")
    source = os.path.join(build.CSRC, "fastcall.cpp")
    (tmp_path / "probe.cpp").write_text(PROBE % source)
    command = [str(tmp_path / "probe.cpp") if a == source else str(tmp_path / "_probe.so") if a == build.FASTCALL else a for a in command]
    subprocess.run(command, check=True)
    r = subprocess.run([sys.executable, "-c", PROGRAM, str(tmp_path)], capture_output=True, text=True, timeout=120)
    assert r.stdout == "leaving\n"
    assert r.returncode == 0, r.stderr
