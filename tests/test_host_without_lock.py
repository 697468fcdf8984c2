"""CPU-only test of csrc/python/without_lock.h: a library call that throws ends in a Python error, with the interpreter lock held and the call
made once."""
import os
import subprocess
import sys
import sysconfig

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MODULE = r"""
#include "without_lock.h"
#include <stdexcept>
static int made = 0;
static int entry(long kind)
{
    ++made;
    if (PyGILState_Check()) return -1;
    if (kind == 1) throw std::bad_alloc();
    if (kind == 2) throw std::length_error("too long");
    if (kind == 3) throw 5;
    return 7;
}
static PyObject *run(PyObject *, PyObject *arg)
{
    const long kind = PyLong_AsLong(arg);
    PyObject *r = without_lock([&] { return entry(kind); });
    if (!PyGILState_Check()) abort();
    return r;
}
static PyObject *calls(PyObject *, PyObject *) { return PyLong_FromLong(made); }
static PyMethodDef methods[] = {{"run", run, METH_O, nullptr}, {"calls", calls, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "locktest", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_locktest(void) { return PyModule_Create(&module); }
"""

PROGRAM = r"""
import locktest, threading, time
print(locktest.run(0))
for kind in (1, 2, 3):
    try:
        print("returned", locktest.run(kind))
    except Exception as e:
        print(type(e).__name__, e)
print(locktest.calls())
going = [True]
def spin():
    while going[0]:
        pass
t = threading.Thread(target=spin)
t.start()
for _ in range(50):                       # with another thread that wants the lock
    try:
        locktest.run(2)
    except RuntimeError:
        pass
going[0] = False
t.join()
print("done")
"""


def test_exceptions_of_a_library_call_reach_python(tmp_path):
    (tmp_path / "m.cpp").write_text(MODULE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fPIC", "-shared", "-I", os.path.join(ROOT, "paper_2507_11978_amd", "csrc", "python"),
                    "-isystem", sysconfig.get_paths()["include"], "m.cpp", "-o", "locktest.so"], cwd=tmp_path, check=True)
    out = subprocess.run([sys.executable, "-c", PROGRAM], cwd=tmp_path, capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stderr
    assert out.stdout.split("\n")[:-1] == ["7", "MemoryError ", "RuntimeError too long", "RuntimeError unknown C++ exception", "4", "done"]
