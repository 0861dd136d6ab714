"""Where C++ exceptions end in the binding's calls (csrc/apmm_call_guard.h), built into a small module of its own: an exception of the body ends there,
and a daemon thread that is ended inside the body, when the interpreter shuts down, does not take the process with it."""
import os
import shutil
import subprocess
import sys
import sysconfig

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_17870_amd", "csrc")

MODULE = r"""
#include <Python.h>
#include <unistd.h>
#include <stdexcept>
#include "apmm_call_guard.h"

// the structure of a call: the interpreter's lock is given back and taken again inside the body
static PyObject *call(PyObject *, PyObject *throws)
{
    const int r = end_exceptions(
        [&] {
            int status;
            Py_BEGIN_ALLOW_THREADS
            status = end_exceptions([] { usleep(50); return 1; }, [] { return 2; });
            Py_END_ALLOW_THREADS
            if (throws == Py_True) throw std::runtime_error("");
            return status;
        },
        [] { return 0; });
    return PyLong_FromLong(r);
}
// checked(check, status), a negative one thrown
static PyObject *checked(PyObject *, PyObject *args)
{
    PyObject *check;
    int status;
    if (!PyArg_ParseTuple(args, "Oi", &check, &status)) return nullptr;
    if (!call_and_check(check, [&] { return status < 0 ? throw std::runtime_error("") : status; })) return nullptr;
    Py_RETURN_TRUE;
}
static PyMethodDef methods[] = {{"call", call, METH_O, nullptr}, {"checked", checked, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "guarded", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_guarded() { return PyModule_Create(&module); }
"""

LOAD = """
import importlib.machinery, importlib.util
loader = importlib.machinery.ExtensionFileLoader("guarded", %r)
guarded = importlib.util.module_from_spec(importlib.util.spec_from_loader("guarded", loader))
"""


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("guard")
    (d / "guarded.cpp").write_text(MODULE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-isystem", sysconfig.get_paths()["include"], "-I", CSRC, str(d / "guarded.cpp"), "-o",
                    str(d / "guarded.so")], check=True, capture_output=True)
    return str(d / "guarded.so")


def test_exceptions_end(library):
    space = {}
    exec(LOAD % library, space)
    assert space["guarded"].call(False) == 1 and space["guarded"].call(True) == 0


def test_status_and_exception_of_a_call(library):
    space = {}
    exec(LOAD % library, space)
    checked, seen = space["guarded"].checked, []

    def check(status):
        seen.append(status)
        if status == 3:
            raise KeyError(status)

    assert checked(check, 0) is True and seen == []
    with pytest.raises(KeyError):
        checked(check, 3)
    with pytest.raises(RuntimeError, match="a call failed"):
        checked(check, 5)
    assert seen == [3, 5]
    with pytest.raises(RuntimeError, match="exception"):  # its own text: the library's last error belongs to another call
        checked(check, -7)
    assert seen == [3, 5]


def test_daemon_threads_at_exit(library):
    program = LOAD % library + """
import threading, time
def loop():
    while True:
        guarded.call(False)
for _ in range(8):
    threading.Thread(target=loop, daemon=True).start()
time.sleep(0.2)
"""
    for _ in range(5):
        r = subprocess.run([sys.executable, "-c", program], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, (r.returncode, r.stderr)


def test_no_other_handler():
    source = open(os.path.join(CSRC, "apmm_call.cpp")).read()
    assert "end_exceptions(" in source and "call_and_check(" in source and "catch" not in source
