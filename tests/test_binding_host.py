"""What the Python binding refuses, keeps and needs before any kernel is launched (no GPU needed)."""
import os
import shutil
import subprocess
import sys
import sysconfig

import pytest

from paper_2309_04875_amd import build, hb


class _Everything:
    """Short cuts that would serve whatever they are given."""
    def __getattr__(self, name):
        return lambda *args: 7


@pytest.mark.parametrize("call", [hb.hb_relu_batch_ex, hb.hb_drelu_batch_ex])
def test_a_batch_without_its_layout_is_refused(call, monkeypatch):
    monkeypatch.setattr(hb, "_native", _Everything())
    monkeypatch.setattr(hb, "_stream_handle", lambda stream: None)
    assert call([], hb.HB_DEALER_PER_GATE) == 7
    with pytest.raises(TypeError):
        call([], None)


THROWING = r"""
#include "hb_gil.hpp"
#include <new>
static PyObject *held_after_throw(PyObject *, PyObject *)
{
    int held = -1;
    try {
        without_gil([]() -> int { throw std::bad_alloc(); });
    } catch (const std::exception &) {
        held = PyGILState_Check();
        if (!held) _exit(3);
    }
    return PyLong_FromLong(held);
}
static PyMethodDef methods[] = {{"held_after_throw", held_after_throw, METH_NOARGS, ""}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "throwing", "", -1, methods, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_throwing() { return PyModule_Create(&module); }
"""


def test_the_interpreter_lock_is_held_where_an_exception_is_caught(tmp_path):
    headers = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(headers, "Python.h")) or shutil.which("g++") is None:
        pytest.skip("needs g++ and Python's headers")
    (tmp_path / "throwing.cpp").write_text("#include <unistd.h>\n" + THROWING)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + headers, "-I" + build.CSRC, str(tmp_path / "throwing.cpp"),
                    "-o", str(tmp_path / "throwing.so")], check=True)
    child = subprocess.run([sys.executable, "-c", "import throwing; assert throwing.held_after_throw() == 1"], cwd=tmp_path, timeout=60)
    assert child.returncode == 0
