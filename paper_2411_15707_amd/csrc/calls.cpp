// The entry points that run per layer, called from Python without ctypes: the arguments of an ordinary call
// (torch tensors on the GPU, ints, a tuple or list of moduli) are checked and handed over here.
// Anything else -- another type, a wrong size, a tensor elsewhere -- is answered None before anything is
// launched, and binding.py goes its own way, which raises what there is to raise.
//
// What it is for: a small call takes the GPU less time than its host.  Of the 5.8 to 6.3 us that a call
// took the host 2.7 were Python's (five attributes of every tensor, the array of moduli, thirteen
// conversions); here they are 0.6.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <limits.h>

#include "../../include/nimbus_cop.h"
#include "../../include/nimbus_rlwe.h"

namespace {

constexpr int kMaxModuli = 8, kMaxBatch = 16;

// the library's entry points (binding.py loads it and hands their addresses over)
struct Entries {
    decltype(&nimbus_cop_matmul) matmul;
    decltype(&nimbus_cop_prepare) prepare;
    decltype(&nimbus_cop_workspace_bytes) workspace_bytes;
    decltype(&nimbus_cop_matmul_prepared) matmul_prepared;
    decltype(&nimbus_cop_stage_shares_batch) stage_shares_batch;
    decltype(&nimbus_cop_matmul_staged_batch) matmul_staged_batch;
    decltype(&nimbus_cop_packed_count) packed_count;
    decltype(&nimbus_cop_pack) pack;
    decltype(&nimbus_rlwe_decrypt) decrypt;
    decltype(&nimbus_rlwe_encrypt) encrypt;
} lib;
PyObject *current_device, *raw_stream;          // torch's, without the Python around them

// The arguments of a call; `ok` turns false at the first that is not the ordinary one.
struct Args {
    PyObject *const *arg;
    Py_ssize_t count;
    bool ok = true;
    uint64_t q[kMaxModuli];

    Args(PyObject *const *args, Py_ssize_t have, Py_ssize_t want) : arg(args), count(have) { ok = have == want; }

    int integer(Py_ssize_t i)                   // positive, below 2^31
    {
        if (!ok || !PyLong_CheckExact(arg[i])) return refuse();
        int overflow = 0;
        const long v = PyLong_AsLongAndOverflow(arg[i], &overflow);
        return overflow || v < 1 || v > INT_MAX ? refuse() : (int)v;
    }
    const uint64_t *moduli(Py_ssize_t i, int L)
    {
        const bool tuple = PyTuple_CheckExact(arg[i]);
        if (!ok || !(tuple || PyList_CheckExact(arg[i]))) return fail();
        const Py_ssize_t n = PySequence_Fast_GET_SIZE(arg[i]);
        if (n < L || n > kMaxModuli) return fail();
        for (Py_ssize_t j = 0; j < n; ++j) {
            PyObject *const item = PySequence_Fast_GET_ITEM(arg[i], j);
            if (!PyLong_CheckExact(item)) return fail();
            q[j] = PyLong_AsUnsignedLongLong(item);
            if (q[j] == (uint64_t)-1) {
                PyErr_Clear();
                return fail();
            }
        }
        return q;
    }
    // a contiguous tensor on the GPU of `items` elements of `size` bytes (items < 0: any number of any size,
    // its bytes to *bytes)
    void *tensor(PyObject *o, __int128 items, int size, size_t *bytes = nullptr)
    {
        if (!ok || !THPVariable_CheckExact(o)) return fail();
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || !t.is_contiguous())
            return fail();
        if (items >= 0 && ((__int128)t.numel() != items || t.element_size() != size)) return fail();
        if (bytes) *bytes = (size_t)t.numel() * (size_t)t.element_size();
        try {
            return t.data_ptr();
        } catch (...) {
            return fail();
        }
    }
    uint64_t *words(Py_ssize_t i, __int128 items) { return ok ? (uint64_t *)tensor(arg[i], items, 8) : fail(); }
    uint64_t *words_or_none(Py_ssize_t i, __int128 items) { return ok && arg[i] != Py_None ? words(i, items) : nullptr; }
    void *bytes(Py_ssize_t i, size_t *size = nullptr) { return ok ? tensor(arg[i], -1, 1, size) : fail(); }
    // a list or tuple of `n` tensors
    template <typename T>
    bool tensors(Py_ssize_t i, int n, __int128 items, T **out, size_t *least = nullptr)
    {
        if (!ok || !(PyTuple_CheckExact(arg[i]) || PyList_CheckExact(arg[i])) || PySequence_Fast_GET_SIZE(arg[i]) != n)
            return refuse() != 0;
        for (int j = 0; j < n; ++j) {
            size_t size = 0;
            out[j] = (T *)tensor(PySequence_Fast_GET_ITEM(arg[i], j), items, items < 0 ? 1 : 8, &size);
            if (least && (j == 0 || size < *least)) *least = size;
        }
        return ok;
    }
    void *stream(Py_ssize_t i)
    {
        if (!ok) return nullptr;
        void *s = nullptr;
        if (PyLong_CheckExact(arg[i])) {
            s = PyLong_AsVoidPtr(arg[i]);
        } else if (arg[i] == Py_None) {
            PyObject *const device = PyObject_CallNoArgs(current_device);
            PyObject *const handle = device ? PyObject_CallOneArg(raw_stream, device) : nullptr;
            if (handle) s = PyLong_AsVoidPtr(handle);
            Py_XDECREF(device);
            Py_XDECREF(handle);
        } else {
            return fail();
        }
        if (PyErr_Occurred()) {
            PyErr_Clear();
            return fail();
        }
        return s;
    }
    int refuse()
    {
        ok = false;
        return 0;
    }
    uint64_t *fail()
    {
        ok = false;
        return nullptr;
    }
};

__int128 columns(int n, int N, int L) { return (__int128)(((long long)n + N - 1) / N) * 2 * L * N; }

// the call itself, without the interpreter's lock; its status, or None where the arguments were not for us
template <typename Call>
PyObject *launch(const Args &a, Call call)
{
    if (!a.ok) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyObject *matmul(PyObject *, PyObject *const *args, Py_ssize_t have)
{
    Args a(args, have, 12);
    const int m = a.integer(1), k = a.integer(2), xb = a.integer(3), n = a.integer(5), N = a.integer(6), L = a.integer(7);
    if (!a.ok) Py_RETURN_NONE;
    const __int128 C = columns(n, N, L);
    const uint64_t *const X = a.words(0, (__int128)m * k), *const ctW = a.words(4, k * C), *const q = a.moduli(8, L),
                   *const mask = a.words_or_none(9, m * C);
    uint64_t *const out = a.words(10, m * C);
    void *const s = a.stream(11);
    return launch(a, [&]() { return lib.matmul(X, m, k, xb, ctW, n, N, L, q, mask, out, s); });
}

PyObject *prepare(PyObject *, PyObject *const *args, Py_ssize_t have)
{
    Args a(args, have, 8);
    const int k = a.integer(1), n = a.integer(2), N = a.integer(3), L = a.integer(4);
    if (!a.ok) Py_RETURN_NONE;
    size_t size = 0;
    const uint64_t *const ctW = a.words(0, k * columns(n, N, L)), *const q = a.moduli(5, L);
    void *const prepared = a.bytes(6, &size), *const s = a.stream(7);
    return launch(a, [&]() { return lib.prepare(ctW, k, n, N, L, q, prepared, size, s); });
}

PyObject *matmul_prepared(PyObject *, PyObject *const *args, Py_ssize_t have)
{
    Args a(args, have, 13);
    const int m = a.integer(1), k = a.integer(2), xb = a.integer(3), n = a.integer(5), N = a.integer(6), L = a.integer(7);
    if (!a.ok) Py_RETURN_NONE;
    const __int128 C = columns(n, N, L);
    size_t size = 0;
    const uint64_t *const X = a.words(0, (__int128)m * k), *const q = a.moduli(8, L), *const mask = a.words_or_none(9, m * C);
    const void *const prepared = a.bytes(4);
    uint64_t *const out = a.words(10, m * C);
    void *const ws = a.bytes(11, &size), *const s = a.stream(12);
    return launch(a, [&]() { return lib.matmul_prepared(X, m, k, xb, prepared, n, N, L, q, mask, out, ws, size, s); });
}

PyObject *stage_shares_batch(PyObject *, PyObject *const *args, Py_ssize_t have)
{
    Args a(args, have, 6);
    const int m = a.integer(1), k = a.integer(2), xb = a.integer(3);
    if (!a.ok || !PyList_CheckExact(args[0]) || PyList_GET_SIZE(args[0]) < 1 || PyList_GET_SIZE(args[0]) > kMaxBatch)
        Py_RETURN_NONE;
    const int count = (int)PyList_GET_SIZE(args[0]);
    const uint64_t *X[kMaxBatch];
    void *ws[kMaxBatch];
    size_t size = 0;
    a.tensors(0, count, (__int128)m * k, X);
    a.tensors(4, count, -1, ws, &size);
    void *const s = a.stream(5);
    return launch(a, [&]() { return lib.stage_shares_batch(count, X, m, k, xb, ws, size, s); });
}

PyObject *matmul_staged_batch(PyObject *, PyObject *const *args, Py_ssize_t have)
{
    Args a(args, have, 12);
    const int m = a.integer(1), k = a.integer(2), xb = a.integer(3), n = a.integer(5), N = a.integer(6), L = a.integer(7);
    if (!a.ok || !PyList_CheckExact(args[10]) || PyList_GET_SIZE(args[10]) < 1 || PyList_GET_SIZE(args[10]) > kMaxBatch)
        Py_RETURN_NONE;
    const int count = (int)PyList_GET_SIZE(args[10]);
    const __int128 C = columns(n, N, L);
    const void *staged[kMaxBatch], *prepared[kMaxBatch];
    const uint64_t *masks[kMaxBatch];
    uint64_t *outs[kMaxBatch];
    size_t size = 0;
    a.tensors(0, count, -1, staged, &size);
    a.tensors(4, count, -1, prepared);
    const uint64_t *const q = a.moduli(8, L);
    const bool masked = args[9] != Py_None;
    if (masked) a.tensors(9, count, m * C, masks);
    a.tensors(10, count, m * C, outs);
    void *const s = a.stream(11);
    if (!a.ok || size < lib.workspace_bytes(m, k, xb)) Py_RETURN_NONE;
    return launch(a, [&]() {
        return lib.matmul_staged_batch(count, staged, m, k, xb, prepared, n, N, L, q, masked ? masks : nullptr, outs, s);
    });
}

PyObject *pack(PyObject *, PyObject *const *args, Py_ssize_t have)
{
    Args a(args, have, 9);
    const int m = a.integer(1), n = a.integer(2), N = a.integer(3), L = a.integer(4);
    if (!a.ok) Py_RETURN_NONE;
    const int T = lib.packed_count(m, n, N);
    if (T < 1) Py_RETURN_NONE;
    const __int128 row = (__int128)2 * L * N;
    const uint64_t *const rows = a.words(0, m * row), *const q = a.moduli(5, L), *const mask = a.words_or_none(6, T * row);
    uint64_t *const packed = a.words(7, T * row);
    void *const s = a.stream(8);
    return launch(a, [&]() { return lib.pack(rows, m, n, N, L, q, mask, packed, s); });
}

PyObject *decrypt(PyObject *, PyObject *const *args, Py_ssize_t have)
{
    Args a(args, have, 10);
    const int T = a.integer(1), N = a.integer(2), L = a.integer(3), tb = a.integer(5);
    if (!a.ok) Py_RETURN_NONE;
    const __int128 words = (__int128)T * N;
    const uint64_t *const ct = a.words(0, words * 2 * L), *const q = a.moduli(4, L);
    const void *const tables = a.bytes(6);
    uint64_t *const phi = a.words(7, words * L), *const m_hat = a.words(8, words);
    void *const s = a.stream(9);
    return launch(a, [&]() { return lib.decrypt(ct, T, N, L, q, tb, tables, phi, m_hat, s); });
}

PyObject *encrypt(PyObject *, PyObject *const *args, Py_ssize_t have)
{
    Args a(args, have, 12);
    const int k = a.integer(1), n = a.integer(2), tb = a.integer(3), N = a.integer(4), L = a.integer(5);
    if (!a.ok) Py_RETURN_NONE;
    const __int128 poly = columns(n, N, L) / (2 * L) * k;           // k Ch N
    const uint64_t *const W = a.words(0, (__int128)k * n), *const q = a.moduli(6, L), *const ap = a.words(8, poly * L);
    const void *const tables = a.bytes(7);
    const int8_t *const e = a.ok ? (const int8_t *)a.tensor(args[9], poly, 1) : nullptr;
    uint64_t *const ctW = a.words(10, poly * 2 * L);
    void *const s = a.stream(11);
    return launch(a, [&]() { return lib.encrypt(W, k, n, tb, N, L, q, tables, ap, e, ctW, s); });
}

// bind(addresses, current_device, raw_stream): addresses in the order of Entries
PyObject *bind(PyObject *, PyObject *args)
{
    PyObject *list, *device, *raw;
    if (!PyArg_ParseTuple(args, "O!OO", &PyTuple_Type, &list, &device, &raw)) return nullptr;
    void *address[sizeof(lib) / sizeof(void *)];
    const Py_ssize_t count = (Py_ssize_t)(sizeof(lib) / sizeof(void *));
    if (PyTuple_GET_SIZE(list) != count) {
        PyErr_SetString(PyExc_ValueError, "one address per entry point");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < count; ++i) {
        address[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(list, i));
        if (!address[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "an entry point without an address");
            return nullptr;
        }
    }
    memcpy(&lib, address, sizeof(lib));
    Py_INCREF(device);
    Py_INCREF(raw);
    Py_XDECREF(current_device);
    Py_XDECREF(raw_stream);
    current_device = device;
    raw_stream = raw;
    Py_RETURN_NONE;
}

#define NIMBUS_FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    NIMBUS_FAST(matmul), NIMBUS_FAST(prepare), NIMBUS_FAST(matmul_prepared), NIMBUS_FAST(stage_shares_batch),
    NIMBUS_FAST(matmul_staged_batch), NIMBUS_FAST(pack), NIMBUS_FAST(decrypt), NIMBUS_FAST(encrypt),
    {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch_version: the torch whose tensors this file was compiled to look into (binding.py compares it)
PyMODINIT_FUNC PyInit__calls(void)
{
    PyObject *const m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", NIMBUS_TORCH_VERSION) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
