"""What the Python binding refuses, keeps and needs before any kernel is launched (no GPU needed)."""
import os
import shutil
import subprocess
import sys
import sysconfig

import pytest

from paper_2309_04875_amd import build, hb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


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


# Allocations of just the armed size fail: 4093 descriptors make plan_launches ask for 4093 bytes.
FAILING = r"""
#include <cstdlib>
#include <new>
static volatile size_t refused = 0;
extern "C" void refuse(size_t bytes) { refused = bytes; }
void *operator new(size_t bytes)
{
    void *p = bytes != 0 && bytes == refused ? nullptr : std::malloc(bytes ? bytes : 1);
    if (p == nullptr) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
"""

NO_MEMORY = r"""
import ctypes, sys
stub = ctypes.CDLL(sys.argv[2], ctypes.RTLD_GLOBAL)          # first, so that the library's operator new is this one
lib = ctypes.CDLL(sys.argv[1])
class Tensor(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("s0", "s1", "o0", "o1")] + [("n", ctypes.c_size_t), ("k", ctypes.c_int), ("m", ctypes.c_int), ("seed", ctypes.c_uint64)]
count = ctypes.c_size_t(4093)
set_ = (Tensor * 4093)(*[Tensor(k=12, m=20) for _ in range(4093)])
bits, plan = ctypes.c_uint64(99), ctypes.c_void_p(99)
stub.refuse(ctypes.c_size_t(4093))
batch = lib.hb_relu_batch(set_, count, ctypes.byref(bits), None)
made = lib.hb_plan_create(set_, count, 1, 0, ctypes.byref(plan))
stub.refuse(ctypes.c_size_t(0))
lib.hb_last_hip_error.restype = ctypes.c_char_p
assert (batch, made) == (-3, -3), (batch, made)
assert bits.value == 99 and plan.value is None and b"memory" in lib.hb_last_hip_error()
assert lib.hb_relu_batch(set_, count, ctypes.byref(bits), None) == 0 and bits.value == 0
"""


def test_no_exception_leaves_the_c_interface(tmp_path):
    if not os.path.exists(hb.LIBRARY) or shutil.which("g++") is None:
        pytest.skip("needs g++ and a built library")
    (tmp_path / "failing.cpp").write_text(FAILING)
    stub = str(tmp_path / "failing.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", str(tmp_path / "failing.cpp"), "-o", stub], check=True)
    child = subprocess.run([sys.executable, "-c", NO_MEMORY, hb.LIBRARY, stub], cwd=tmp_path, timeout=120,
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert child.returncode == 0, child.stdout


def test_functions_of_numbers_need_no_torch():
    child = subprocess.run([sys.executable, "-W", "error", "-c", "import sys; sys.modules['torch'] = None\nfrom paper_2309_04875_amd import hb\n"
                            "print(hb.hb_tensor_seed(1, 2), hb.hb_opened_bits(1, 12, 20, 1000), hb.hb_party_workspace_bytes(100, 12, 20))"],
                           cwd=ROOT, timeout=120, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert child.returncode == 0, child.stdout
    assert child.stdout.split() == [str(v) for v in (hb.hb_tensor_seed(1, 2), hb.hb_opened_bits(1, 12, 20, 1000), hb.hb_party_workspace_bytes(100, 12, 20))]


def test_calls_go_through_ctypes_without_the_native_binding(monkeypatch):
    hb.load()
    name = hb.__package__ + "._binding"
    monkeypatch.delattr(sys.modules[hb.__package__], "_binding", raising=False)
    monkeypatch.setitem(sys.modules, name, None)                       # cannot be imported
    monkeypatch.setattr(hb, "_native", hb._NotLoaded)
    with pytest.warns(UserWarning, match="ctypes"):
        assert hb._native.shares(1, None, None, 12, 20, 1, None, None, None) is NotImplemented
    assert hb._native is hb._NotThere and hb._native.batch(1, [], None) is NotImplemented


def test_build_without_python_headers(monkeypatch, tmp_path, capsys):
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    monkeypatch.setattr(build, "BINDING", str(tmp_path / "_binding.so"))
    (tmp_path / "_binding.so").write_text("of an older build")
    build._build_binding()
    assert "Python.h" in capsys.readouterr().out and not (tmp_path / "_binding.so").exists()


def test_the_binding_calls_the_library_beside_it(tmp_path):
    """Another libhb.so in LD_LIBRARY_PATH, here one without functions, is not what `_binding` takes."""
    if not os.path.exists(hb.BINDING) or shutil.which("gcc") is None:
        pytest.skip("needs gcc and a built binding")
    (tmp_path / "empty.c").write_text("int nothing;\n")
    subprocess.run(["gcc", "-shared", "-fPIC", str(tmp_path / "empty.c"), "-o", str(tmp_path / "libhb.so")], check=True)
    path = str(tmp_path) + os.pathsep + os.environ.get("LD_LIBRARY_PATH", "")
    child = subprocess.run([sys.executable, "-W", "error", "-c", "import torch; from paper_2309_04875_amd import hb; hb.load()\n"
                            "assert hb._native.__name__.endswith('_binding')\n"
                            "with open('/proc/self/maps') as maps: print({l.split()[-1] for l in maps if l.rstrip().endswith('libhb.so')})"],
                           cwd=ROOT, env=dict(os.environ, LD_LIBRARY_PATH=path), timeout=120, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert child.returncode == 0 and child.stdout.strip() == str({os.path.realpath(hb.LIBRARY)}), child.stdout
