"""A library call that throws while the interpreter's lock is released has taken it again by the time the error
is turned into a Python one.  Compiled and run in a process of its own: without the lock that process dies."""
import os
import subprocess
import sys
import sysconfig

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_06938_amd", "csrc")

MODULE = r"""
#include "unlocked.hpp"
#include <stdexcept>
static PyObject *call(PyObject *, PyObject *arg)
{
    const long v = PyLong_AsLong(arg);
    try {
        const long r = swimba::unlocked([&] { if (v < 0) throw std::runtime_error("below zero"); return 2 * v; });
        return PyLong_FromLong(r);
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}
static PyMethodDef methods[] = {{"call", call, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "thrower", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_thrower() { return PyModule_Create(&module); }
"""

USE = r"""
import threading, thrower
for _ in range(3):
    try:
        thrower.call(-1)
    except RuntimeError as e:
        assert str(e) == "below zero"
    else:
        raise AssertionError("not raised")
t = threading.Thread(target=thrower.call, args=(1,))
t.start(); t.join()
assert thrower.call(4) == 8
print("held")
"""


def test_the_lock_is_held_again_after_a_throw(tmp_path):
    (tmp_path / "thrower.cpp").write_text(MODULE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + sysconfig.get_paths()["include"], "-I" + CSRC,
                    str(tmp_path / "thrower.cpp"), "-o", str(tmp_path / "thrower.so")], check=True)
    r = subprocess.run([sys.executable, "-c", USE], cwd=tmp_path, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "held", (r.returncode, r.stderr[-500:])
