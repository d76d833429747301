// The binding's two short calls, prefill and decode step, from Python objects to the C entry points without an interpreter between: a prompt
// of a few hundred rows is one launch of 10 us, and checks, sizes, pointers and four buffers in Python were 9 of the 13 us that the host took.
// Only calls that are in order are made here.  Whatever else is passed in is answered with None, and the binding's Python code takes the call
// and says what is wrong with it; a status other than 0 comes back as a number.
#include <Python.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>

#include <limits.h>
#include <stdint.h>

#include "../../include/delta_attn.h"

namespace {

// the library's entry points, as the binding has loaded them
decltype(&delta_attn_prefill) prefill_entry = nullptr;
decltype(&delta_attn_prefill_workspace_bytes) workspace_entry = nullptr;
decltype(&delta_attn_decode) decode_entry = nullptr;

PyObject *not_here() { Py_RETURN_NONE; }

// A plain tensor (or parameter) on a GPU, contiguous, of `dims` sizes of at most 31 bits; else NULL.
const at::Tensor *tensor(PyObject *o, int64_t dims) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.dim() != dims || !t.is_contiguous()) return nullptr;
    for (const int64_t s : t.sizes())
        if (s > INT32_MAX) return nullptr;
    return &t;
}
// whether its strides are those that torch gives a new tensor (those of sizes of 1 are otherwise free, and torch.empty_like keeps them)
bool usual_strides(const at::Tensor &t) {
    int64_t want = 1;
    for (int64_t k = t.dim() - 1; k >= 0; --k) {
        if (t.stride(k) != want) return false;
        want *= t.size(k) > 1 ? t.size(k) : 1;
    }
    return true;
}
bool number(PyObject *o, int32_t *to) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || v < INT32_MIN || v > INT32_MAX) return false;
    *to = (int32_t)v;
    return true;
}
bool number(PyObject *o, float *to) {
    if (!PyFloat_CheckExact(o)) return false;
    *to = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
// a buffer that the caller passes in, as it is: NULL where it is no tensor
const at::Tensor *buffer(PyObject *o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

int dtype_of(const at::Tensor &t) {
    return t.scalar_type() == at::kFloat ? DA_F32 : t.scalar_type() == at::kBFloat16 ? DA_BF16 : -1;
}
void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }
// The interpreter's lock is given back while one of these lives: an allocation may wait for the device, and so for a host function on a
// stream that wants the lock.
struct Unlocked {
    PyThreadState *const state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// prefill(Q, K, V, theta, window, scale, score_mode, window_mode, cache's handle, workspace, out)
PyObject *prefill(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    if (!prefill_entry || count != 11) return not_here();
    const at::Tensor *Q = tensor(args[0], 4), *K = tensor(args[1], 4), *V = tensor(args[2], 4);
    da_prefill_params p;
    if (!Q || !K || !V || !number(args[3], &p.theta) || !number(args[4], &p.window) || !number(args[5], &p.scale)) return not_here();
    int32_t score_mode, window_mode;
    if (!number(args[6], &score_mode) || !number(args[7], &window_mode) || !PyLong_CheckExact(args[8])) return not_here();
    p.score_mode = decltype(p.score_mode)(score_mode);
    p.window_mode = decltype(p.window_mode)(window_mode);
    const int dtype = dtype_of(*K);
    if (dtype < 0 || Q->scalar_type() != K->scalar_type() || V->scalar_type() != K->scalar_type() || V->sizes() != K->sizes() || Q->size(0) != K->size(0) ||
        Q->size(2) != K->size(2) || Q->size(3) != K->size(3))
        return not_here();
    p.dtype = decltype(p.dtype)(dtype);
    p.batch = (int32_t)Q->size(0);
    p.n_q_heads = (int32_t)Q->size(1);
    p.n_kv_heads = (int32_t)K->size(1);
    p.seq_len = (int32_t)Q->size(2);
    p.head_dim = (int32_t)Q->size(3);
    da_cache *const cache = (da_cache *)PyLong_AsVoidPtr(args[8]);
    if (!cache && PyErr_Occurred()) return nullptr;
    const bool made = args[10] == Py_None;
    const at::Tensor *out[3] = {};
    if (made) {
        if (!usual_strides(*Q)) return not_here();
    } else {
        if (!PyTuple_CheckExact(args[10]) || PyTuple_GET_SIZE(args[10]) != 3) return not_here();
        for (int k = 0; k < 3; ++k)
            if (!(out[k] = buffer(PyTuple_GET_ITEM(args[10], k)))) return not_here();
    }
    const at::Tensor *workspace = nullptr;
    if (args[9] != Py_None && !(workspace = buffer(args[9]))) return not_here();
    at::Tensor room, O, mask, nnz;
    da_status st;
    {
        const Unlocked unlocked;
        if (!workspace) {
            const size_t bytes = workspace_entry(&p);
            room = at::empty({(int64_t)(bytes ? bytes : 1)}, Q->options().dtype(at::kByte));
            workspace = &room;
        }
        if (made) {
            O = at::empty(Q->sizes(), Q->options());
            mask = at::empty({p.batch, p.n_kv_heads, p.seq_len, p.head_dim / 32}, Q->options().dtype(at::kInt));
            nnz = at::empty({p.batch, p.n_kv_heads}, Q->options().dtype(at::kLong));
            out[0] = &O, out[1] = &mask, out[2] = &nnz;
        }
        st = prefill_entry(&p, Q->data_ptr(), K->data_ptr(), V->data_ptr(), out[0]->data_ptr(), (uint32_t *)out[1]->data_ptr(),
                           (uint64_t *)out[2]->data_ptr(), cache, workspace->data_ptr(), (size_t)workspace->numel(), stream());
    }
    if (st != DA_OK) return PyLong_FromLong((long)st);
    PyObject *const result = PyTuple_New(3);
    if (!result) return nullptr;
    for (int i = 0; i < 3; ++i) {
        PyObject *one;
        if (made) {
            one = THPVariable_Wrap(i == 0 ? std::move(O) : i == 1 ? std::move(mask) : std::move(nnz));
        } else {
            one = PyTuple_GET_ITEM(args[10], i);
            Py_INCREF(one);
        }
        if (!one) {
            Py_DECREF(result);
            return nullptr;
        }
        PyTuple_SET_ITEM(result, i, one);
    }
    return result;
    END_HANDLE_TH_ERRORS
}

// what a decode step needs of its cache, packed by the binding (bytes)
struct CacheOf {
    da_cache *handle;
    int32_t batch, n_q_heads, n_kv_heads, head_dim, dtype, none;
};

// decode(CacheOf, q_new, k_new, v_new, out, mask_row)
PyObject *decode(PyObject *, PyObject *const *args, Py_ssize_t count) {
    HANDLE_TH_ERRORS
    if (!decode_entry || count != 6 || !PyBytes_CheckExact(args[0]) || PyBytes_GET_SIZE(args[0]) != (Py_ssize_t)sizeof(CacheOf)) return not_here();
    CacheOf c;
    memcpy(&c, PyBytes_AS_STRING(args[0]), sizeof(c));
    const at::Tensor *q = tensor(args[1], 3), *k = tensor(args[2], 3), *v = tensor(args[3], 3);
    if (!q || !k || !v) return not_here();
    auto fits = [&](const at::Tensor &t, int32_t heads) {
        return t.size(0) == c.batch && t.size(1) == heads && t.size(2) == c.head_dim && dtype_of(t) == c.dtype;
    };
    if (!fits(*q, c.n_q_heads) || !fits(*k, c.n_kv_heads) || !fits(*v, c.n_kv_heads)) return not_here();
    const at::Tensor *out = nullptr, *row = nullptr;
    at::Tensor new_out, new_row;
    if (args[4] != Py_None) {
        if (!(out = buffer(args[4]))) return not_here();
    } else if (!usual_strides(*q)) {
        return not_here();
    }
    if (args[5] != Py_None && !(row = buffer(args[5]))) return not_here();
    da_status st;
    {
        const Unlocked unlocked;
        if (!out) {
            new_out = at::empty(q->sizes(), q->options());
            out = &new_out;
        }
        if (!row) {
            new_row = at::empty({c.batch, c.n_kv_heads, c.head_dim / 32}, q->options().dtype(at::kInt));
            row = &new_row;
        }
        st = decode_entry(c.handle, q->data_ptr(), k->data_ptr(), v->data_ptr(), out->data_ptr(), (uint32_t *)row->data_ptr(), stream());
    }
    if (st != DA_OK) return PyLong_FromLong((long)st);
    PyObject *const a = out == &new_out ? THPVariable_Wrap(std::move(new_out)) : (Py_INCREF(args[4]), args[4]);
    PyObject *const b = row == &new_row ? THPVariable_Wrap(std::move(new_row)) : (Py_INCREF(args[5]), args[5]);
    PyObject *const result = a && b ? PyTuple_New(2) : nullptr;
    if (!result) {
        Py_XDECREF(a);
        Py_XDECREF(b);
        return nullptr;
    }
    PyTuple_SET_ITEM(result, 0, a);
    PyTuple_SET_ITEM(result, 1, b);
    return result;
    END_HANDLE_TH_ERRORS
}

// bind(addresses of delta_attn_prefill, delta_attn_prefill_workspace_bytes, delta_attn_decode)
PyObject *bind(PyObject *, PyObject *args) {
    unsigned long long a, b, c;
    if (!PyArg_ParseTuple(args, "KKK", &a, &b, &c)) return nullptr;
    prefill_entry = (decltype(prefill_entry))(uintptr_t)a;
    workspace_entry = (decltype(workspace_entry))(uintptr_t)b;
    decode_entry = (decltype(decode_entry))(uintptr_t)c;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                         {"prefill", (PyCFunction)(void (*)(void))prefill, METH_FASTCALL, nullptr},
                         {"decode", (PyCFunction)(void (*)(void))decode, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__marshal() {
    PyObject *const m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", BUILT_FOR) < 0) {   // torch.__version__
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
