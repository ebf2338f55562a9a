// Argument marshalling of the Python binding in native code: a CPython module (paper_2309_04875_amd._binding) whose functions
// take torch tensors and call the C ABI of include/hb.h.
//
// What it is for: the calls on small tensors are bound by the host, and of the 6.6 us of one (2^16 elements) 2.5 were
// spent in Python on four tensors' checks and ctypes' conversions; here they take about 0.4.  A batch of 17 tensors of one small image
// was made in 25 us and is in 2.
//
// Every function is a short cut of the Python function of the same purpose in hb.py and returns NotImplemented, having done
// nothing, for whatever it does not know at sight: tensors of a subclass, of another type or device, not contiguous or of
// different sizes, numbers that are not plain ints, a stream of the caller's, outputs left out.  The Python function then
// goes on as if it had not been called, and raises what it always raised.
#include <Python.h>

#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <vector>

#include "../../include/hb.h"
#include "hb_gil.hpp"

namespace {

PyObject *g_check = nullptr;      // hb._check: raises the exception of a status

PyObject *not_known() { Py_RETURN_NOTIMPLEMENTED; }

const at::Tensor *tensor_of(PyObject *o, at::ScalarType type)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.scalar_type() == type && t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}

// Tensors of one size, whose addresses go to `at`.
class Tensors {
  public:
    template <class Pointer>
    void take(PyObject *o, at::ScalarType type, Pointer *&at)
    {
        const at::Tensor *t = ok ? tensor_of(o, type) : nullptr;
        ok = t != nullptr && (n < 0 || n == t->numel());
        if (!ok) return;
        n = t->numel();
        at = static_cast<Pointer *>(t->data_ptr());
    }
    bool ok = true;
    int64_t n = -1;
};

// Plain ints, reduced as ctypes and the mask of a seed reduce them.
bool word_of(PyObject *o, uint64_t &v)
{
    if (!PyLong_CheckExact(o)) return false;
    v = PyLong_AsUnsignedLongLongMask(o);
    return true;
}
bool int_of(PyObject *o, int &v)
{
    uint64_t w = 0;
    const bool known = word_of(o, w);
    v = (int)(uint32_t)w;
    return known;
}

void *current_stream() { return c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream(); }

// The result of a call, or the exception of its status.
PyObject *checked(int st, PyObject *result)
{
    if (st == HB_OK) return result;
    Py_XDECREF(result);
    PyObject *none = PyObject_CallFunction(g_check, "i", st);
    Py_XDECREF(none);
    return nullptr;                       // hb._check has raised
}

// Runs `body`, which returns what the function returns; C++ exceptions (tensors without memory of their own) are left to the
// Python function.  They come from before the C call, which throws none, and nothing after it does.
template <class Body>
PyObject *guarded(const Body &body)
{
    try {
        return body();
    } catch (const std::exception &) {
        PyErr_Clear();                    // where the exception came out of Python code (a dispatch mode of torch)
        return not_known();
    }
}

using SharesCall = int (*)(const int64_t *, const int64_t *, size_t, int, int, uint64_t, int64_t *, int64_t *, uint64_t *, void *);
using SharesCallEx = int (*)(const int64_t *, const int64_t *, size_t, int, int, uint64_t, int, int64_t *, int64_t *, uint64_t *, void *);

// shares(which, share0, share1, k, m, seed, dealer or None, out0, out1) -> (out0, out1, opened bits)
PyObject *shares(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    static const SharesCall plain[] = {hb_drelu, hb_relu, hb_sign_shares};
    static const SharesCallEx ex[] = {hb_drelu_ex, hb_relu_ex};
    return guarded([&]() -> PyObject * {
        int which = -1, k = 0, m = 0, dealer = 0;
        uint64_t seed = 0, bits = 0;
        if (count != 9 || !int_of(a[0], which) || !int_of(a[3], k) || !int_of(a[4], m) || !word_of(a[5], seed)) return not_known();
        const bool has_dealer = a[6] != Py_None;
        if (which < 0 || which >= (has_dealer ? 2 : 3) || (has_dealer && !int_of(a[6], dealer))) return not_known();
        const int64_t *s0 = nullptr, *s1 = nullptr;
        int64_t *o0 = nullptr, *o1 = nullptr;
        Tensors t;
        t.take(a[1], at::kLong, s0);
        t.take(a[2], at::kLong, s1);
        t.take(a[7], at::kLong, o0);
        t.take(a[8], at::kLong, o1);
        if (!t.ok) return not_known();
        void *stream = current_stream();
        const int st = without_gil([&] {
            return has_dealer ? ex[which](s0, s1, (size_t)t.n, k, m, seed, dealer, o0, o1, &bits, stream)
                              : plain[which](s0, s1, (size_t)t.n, k, m, seed, o0, o1, &bits, stream);
        });
        return checked(st, st == HB_OK ? Py_BuildValue("OOK", a[7], a[8], (unsigned long long)bits) : nullptr);
    });
}

// parties(relu, shares, k, m, seed, outs) -> opened bits
PyObject *parties(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        constexpr Py_ssize_t kMost = 8;
        int relu = 0, k = 0, m = 0;
        uint64_t seed = 0, bits = 0;
        if (count != 6 || !int_of(a[0], relu) || !int_of(a[2], k) || !int_of(a[3], m) || !word_of(a[4], seed)) return not_known();
        if (!PyList_CheckExact(a[1]) || !PyList_CheckExact(a[5])) return not_known();
        const Py_ssize_t p = PyList_GET_SIZE(a[1]);
        if (p < 1 || p > kMost || PyList_GET_SIZE(a[5]) != p) return not_known();
        const int64_t *in[kMost] = {};
        int64_t *out[kMost] = {};
        Tensors t;
        for (Py_ssize_t q = 0; q < p; ++q) t.take(PyList_GET_ITEM(a[1], q), at::kLong, in[q]);
        for (Py_ssize_t q = 0; q < p; ++q) t.take(PyList_GET_ITEM(a[5], q), at::kLong, out[q]);
        if (!t.ok) return not_known();
        void *stream = current_stream();
        const int st = without_gil([&] { return (relu ? hb_relu_mp : hb_drelu_mp)(in, (int)p, (size_t)t.n, k, m, seed, out, &bits, stream); });
        return checked(st, st == HB_OK ? PyLong_FromUnsignedLongLong(bits) : nullptr);
    });
}

// batch(relu, list of (share0, share1, out0, out1, k, m, seed), dealer or None) -> opened bits
PyObject *batch(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        int relu = 0, dealer = 0;
        if (count != 3 || !int_of(a[0], relu) || (!PyList_CheckExact(a[1]) && !PyTuple_CheckExact(a[1]))) return not_known();
        const bool has_dealer = a[2] != Py_None;
        if (has_dealer && !int_of(a[2], dealer)) return not_known();
        const Py_ssize_t items = PySequence_Fast_GET_SIZE(a[1]);
        std::vector<hb_tensor> set((size_t)items);
        for (Py_ssize_t i = 0; i < items; ++i) {
            PyObject *item = PySequence_Fast_GET_ITEM(a[1], i);
            if (!PyTuple_CheckExact(item) || PyTuple_GET_SIZE(item) != 7) return not_known();
            hb_tensor &d = set[(size_t)i];
            Tensors t;
            t.take(PyTuple_GET_ITEM(item, 0), at::kLong, d.share0);
            t.take(PyTuple_GET_ITEM(item, 1), at::kLong, d.share1);
            t.take(PyTuple_GET_ITEM(item, 2), at::kLong, d.out0);
            t.take(PyTuple_GET_ITEM(item, 3), at::kLong, d.out1);
            if (!t.ok || !int_of(PyTuple_GET_ITEM(item, 4), d.k) || !int_of(PyTuple_GET_ITEM(item, 5), d.m) ||
                !word_of(PyTuple_GET_ITEM(item, 6), d.seed))
                return not_known();
            d.n = (size_t)t.n;
        }
        uint64_t bits = 0;
        void *stream = current_stream();
        const int st = without_gil([&] {
            if (has_dealer) return (relu ? hb_relu_batch_ex : hb_drelu_batch_ex)(set.data(), set.size(), dealer, &bits, stream);
            return (relu ? hb_relu_batch : hb_drelu_batch)(set.data(), set.size(), &bits, stream);
        });
        return checked(st, st == HB_OK ? PyLong_FromUnsignedLongLong(bits) : nullptr);
    });
}

// plan_run(address of the plan) -> opened bits
PyObject *plan_run(PyObject *, PyObject *plan)
{
    return guarded([&]() -> PyObject * {
        uint64_t address = 0, bits = 0;
        if (!word_of(plan, address) || address == 0) return not_known();
        void *stream = current_stream();
        const int st = without_gil([&] { return hb_plan_run(reinterpret_cast<const hb_plan *>(address), &bits, stream); });
        return checked(st, st == HB_OK ? PyLong_FromUnsignedLongLong(bits) : nullptr);
    });
}

PyObject *given(PyObject *o)
{
    Py_INCREF(o);
    return o;
}

// sim_relu(x, k, m, seed, share_seed, out) -> out
PyObject *sim_relu(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        int k = 0, m = 0;
        uint64_t seed = 0, share_seed = 0;
        if (count != 6 || !int_of(a[1], k) || !int_of(a[2], m) || !word_of(a[3], seed) || !word_of(a[4], share_seed)) return not_known();
        const float *x = nullptr;
        float *y = nullptr;
        Tensors t;
        t.take(a[0], at::kFloat, x);
        t.take(a[5], at::kFloat, y);
        if (!t.ok) return not_known();
        void *stream = current_stream();
        const int st = without_gil([&] { return hb_sim_relu_f32(x, (size_t)t.n, k, m, seed, share_seed, y, stream); });
        return checked(st, st == HB_OK ? given(a[5]) : nullptr);
    });
}

// share(x, share_seed, share0, share1) -> (share0, share1)
PyObject *share(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        uint64_t seed = 0;
        if (count != 4 || !word_of(a[1], seed)) return not_known();
        const float *x = nullptr;
        int64_t *s0 = nullptr, *s1 = nullptr;
        Tensors t;
        t.take(a[0], at::kFloat, x);
        t.take(a[2], at::kLong, s0);
        t.take(a[3], at::kLong, s1);
        if (!t.ok) return not_known();
        void *stream = current_stream();
        const int st = without_gil([&] { return hb_share_f32(x, (size_t)t.n, seed, s0, s1, stream); });
        return checked(st, st == HB_OK ? PyTuple_Pack(2, a[2], a[3]) : nullptr);
    });
}

// reveal(share0, share1, out) -> out
PyObject *reveal(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        if (count != 3) return not_known();
        const int64_t *s0 = nullptr, *s1 = nullptr;
        float *y = nullptr;
        Tensors t;
        t.take(a[0], at::kLong, s0);
        t.take(a[1], at::kLong, s1);
        t.take(a[2], at::kFloat, y);
        if (!t.ok) return not_known();
        void *stream = current_stream();
        const int st = without_gil([&] { return hb_reveal_f32(s0, s1, (size_t)t.n, y, stream); });
        return checked(st, st == HB_OK ? given(a[2]) : nullptr);
    });
}

// eco_scan(share0, share1, counts) -> counts
PyObject *eco_scan(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        if (count != 3) return not_known();
        const int64_t *s0 = nullptr, *s1 = nullptr;
        int64_t *counts = nullptr;
        Tensors t, c;
        t.take(a[0], at::kLong, s0);
        t.take(a[1], at::kLong, s1);
        c.take(a[2], at::kLong, counts);
        if (!t.ok || !c.ok || c.n != 64) return not_known();
        void *stream = current_stream();
        const int st = without_gil([&] { return hb_eco_scan(s0, s1, (size_t)t.n, reinterpret_cast<uint64_t *>(counts), stream); });
        return checked(st, st == HB_OK ? given(a[2]) : nullptr);
    });
}

// party(share0, share1, k, m, seed, dealer or None, out0, out1, workspace) -> (out0, out1, wire 0, wire 1, wire bytes)
PyObject *party(PyObject *, PyObject *const *a, Py_ssize_t count)
{
    return guarded([&]() -> PyObject * {
        int k = 0, m = 0, dealer = 0;
        uint64_t seed = 0, bytes = 0;
        if (count != 9 || !int_of(a[2], k) || !int_of(a[3], m) || !word_of(a[4], seed)) return not_known();
        const bool has_dealer = a[5] != Py_None;
        if (has_dealer && !int_of(a[5], dealer)) return not_known();
        const int64_t *s0 = nullptr, *s1 = nullptr;
        int64_t *o0 = nullptr, *o1 = nullptr;
        Tensors t;
        t.take(a[0], at::kLong, s0);
        t.take(a[1], at::kLong, s1);
        t.take(a[6], at::kLong, o0);
        t.take(a[7], at::kLong, o1);
        const at::Tensor *workspace = tensor_of(a[8], at::kByte);
        if (!t.ok || workspace == nullptr || workspace->dim() != 1) return not_known();
        const size_t n = (size_t)t.n, workspace_bytes = (size_t)workspace->numel();
        // The views of the wires are made before the launch: what throws here has not been enqueued and may be left to the Python
        // function, which would enqueue it a second time otherwise.
        const int64_t words = (int64_t)(has_dealer ? hb_party_wire_words_ex(n, k, m, dealer) : hb_party_wire_words(n, k, m));
        THPObjectPtr wires[2];
        for (int p = 0; p < 2; ++p) {
            const int64_t at = (int64_t)(has_dealer ? hb_party_wire_offset_ex(n, k, m, dealer, p) : hb_party_wire_offset(n, k, m, p));
            wires[p] = THPVariable_Wrap(workspace->slice(0, at, at + 8 * words).view(at::kLong));
        }
        void *to = workspace->data_ptr(), *stream = current_stream();
        const int st = without_gil([&] {
            return has_dealer ? hb_relu_party_ex(s0, s1, n, k, m, seed, dealer, o0, o1, to, workspace_bytes, &bytes, stream)
                              : hb_relu_party(s0, s1, n, k, m, seed, o0, o1, to, workspace_bytes, &bytes, stream);
        });
        if (st != HB_OK) return checked(st, nullptr);
        return Py_BuildValue("OOOOK", a[6], a[7], wires[0].get(), wires[1].get(), (unsigned long long)bytes);
    });
}

PyObject *initialise(PyObject *, PyObject *check)
{
    Py_INCREF(check);
    Py_XDECREF(g_check);
    g_check = check;
    Py_RETURN_NONE;
}

#define HB_FAST(name, doc) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, doc}
PyMethodDef g_methods[] = {
    HB_FAST(shares, "DReLU, ReLU or sign shares of a pair of share tensors"),
    HB_FAST(parties, "DReLU or ReLU among several parties"),
    HB_FAST(batch, "DReLU or ReLU of a set of tensors"),
    HB_FAST(sim_relu, "simulator ReLU of floats"),
    HB_FAST(share, "encode and share floats"),
    HB_FAST(reveal, "open and decode shares"),
    HB_FAST(eco_scan, "zero-error scan"),
    HB_FAST(party, "party-faithful ReLU"),
    {"plan_run", plan_run, METH_O, "enqueue a plan"},
    {"initialise", initialise, METH_O, "the function that raises the exception of a status"},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", "argument marshalling of hb.py", -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding()
{
    PyObject *module = PyModule_Create(&g_module);
    if (module != nullptr && PyModule_AddStringConstant(module, "torch_version", HB_TORCH_VERSION) != 0) Py_CLEAR(module);
    return module;
}
