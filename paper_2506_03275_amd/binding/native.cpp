// The hot entry points of the Python binding without Python in between: a small call took 2.5 us of attribute look-ups on
// its tensors before it reached the library, of the 6 that it took in all, and the smallest kernels take 4.
//
// Each function here takes exactly what the Python function of its name takes, by position.  It answers only the plain
// case (exact torch tensors of the right type and layout, ints and floats) with the library's status; for everything
// else, also for whatever is wrong, it returns None, and the Python function does the whole call itself, with its own
// checks and messages.
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

#include "../../include/chipmunk.h"

namespace {

struct Entry {
    const char* name;
    void* at;
};
Entry entries[] = {{"chipmunk_voxel_reorder", nullptr},       {"chipmunk_topk_cols", nullptr},
                   {"chipmunk_attn_sparse_delta", nullptr},   {"chipmunk_attn_dense", nullptr},
                   {"chipmunk_attn_dense_colsum_stale", nullptr}, {"chipmunk_mlp_tile_mean_preact", nullptr},
                   {"chipmunk_mlp_sparse_delta", nullptr},    {"chipmunk_mlp_dense", nullptr}};
enum { kReorder, kTopk, kAttnDelta, kAttnDense, kAttnRefresh, kScores, kMlpDelta, kMlpDense };
PyObject* current_device = nullptr;   // torch's functions that name the current device and, for a device, its current stream
PyObject* raw_stream = nullptr;

// One call's arguments; ok turns false with the first that the plain case does not cover.
struct Args {
    PyObject* const* v;
    bool ok;

    const at::Tensor* tensor(int i) {
        if (!ok || !THPVariable_CheckExact(v[i])) {
            ok = false;
            return nullptr;
        }
        return &THPVariable_Unpack(v[i]);
    }
    // data of a contiguous GPU tensor of this type; None: null
    void* data(int i, at::ScalarType type) {
        if (!ok || none(i)) return nullptr;
        const at::Tensor* t = tensor(i);
        if (!ok || t->scalar_type() != type || !t->is_cuda() || !t->is_contiguous()) {
            ok = false;
            return nullptr;
        }
        return t->data_ptr();
    }
    const uint16_t* bf16(int i) { return static_cast<const uint16_t*>(data(i, at::kBFloat16)); }
    uint16_t* bf16_out(int i) { return static_cast<uint16_t*>(data(i, at::kBFloat16)); }
    int32_t* i32(int i) { return static_cast<int32_t*>(data(i, at::kInt)); }
    float* f32(int i) { return static_cast<float*>(data(i, at::kFloat)); }
    // size `dim` of a tensor of `dims` dimensions (-1: the last of any)
    int size(int i, int dims, int dim) {
        const at::Tensor* t = tensor(i);
        if (!ok || (dims >= 0 ? t->dim() != dims : t->dim() < 1)) {
            ok = false;
            return 0;
        }
        const int64_t n = t->size(dims >= 0 ? dim : t->dim() - 1);
        if (n > INT_MAX) ok = false;
        return (int)n;
    }
    bool none(int i) const { return v[i] == Py_None; }
    int rows(int i) {          // a tensor's first size
        const at::Tensor* t = tensor(i);
        if (!ok || t->dim() < 1 || t->size(0) > INT_MAX) {
            ok = false;
            return 0;
        }
        return (int)t->size(0);
    }
    size_t elements(int i) {   // None: 0
        if (!ok || none(i)) return 0;
        const at::Tensor* t = tensor(i);
        return ok ? (size_t)t->numel() : 0;
    }
    int integer(int i) {
        if (!ok || !PyLong_CheckExact(v[i])) {
            ok = false;
            return 0;
        }
        int over = 0;
        const long n = PyLong_AsLongAndOverflow(v[i], &over);
        if (over || n > INT_MAX || n < INT_MIN) ok = false;
        return (int)n;
    }
    float real(int i) {
        if (!ok || !PyFloat_CheckExact(v[i])) {
            ok = false;
            return 0.f;
        }
        return (float)PyFloat_AS_DOUBLE(v[i]);
    }
    void* stream() {
        if (!ok) return nullptr;
        PyObject* device = PyObject_CallNoArgs(current_device);
        PyObject* s = device ? PyObject_CallOneArg(raw_stream, device) : nullptr;
        void* at = s ? PyLong_AsVoidPtr(s) : nullptr;
        Py_XDECREF(device);
        Py_XDECREF(s);
        if (PyErr_Occurred()) ok = false;
        return at;
    }
};

// call(a): the library's status, the GIL released around the library itself by `run`, whose first argument only names the
// function's type (a reference to the function itself would need the library at link time)
template <typename Call>
PyObject* answer(int entry, PyObject* const* args, Py_ssize_t n, Py_ssize_t want, Call&& call) {
    if (!entries[entry].at || n != want) Py_RETURN_NONE;
    Args a{args, true};
    int32_t status = 0;
    try {
        call(a, [&](auto f, auto... values) {
            if (!a.ok) return;
            PyThreadState* state = PyEval_SaveThread();
            status = reinterpret_cast<decltype(f)>(entries[entry].at)(values...);
            PyEval_RestoreThread(state);
        });
    } catch (...) {
        a.ok = false;
    }
    if (!a.ok) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(status);
}

// Arguments are read into variables, in order, before the call: a call's own arguments have no order, and `ok` must be
// known.

// src, dst, perm, inv_perm, n_prefix, T, H, W, n_suffix, vt, vh, vw, inverse
PyObject* voxel_reorder(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return answer(kReorder, args, n, 13, [](Args& a, auto run) {
        const at::Tensor *src = a.tensor(0), *dst = a.tensor(1);   // (permutations alone: the Python function)
        if (!a.ok || src->dim() < 2 || src->size(0) < 1 || src->size(1) < 1 || src->sizes() != dst->sizes() || src->size(0) > INT_MAX) {
            a.ok = false;
            return;
        }
        const int64_t row = src->numel() / (src->size(0) * src->size(1)) * (int64_t)src->element_size();
        if (row > INT_MAX || !PyBool_Check(a.v[12])) a.ok = false;
        const void* from = a.data(0, src->scalar_type());
        void* to = a.data(1, src->scalar_type());
        int32_t *perm = a.i32(2), *inv = a.i32(3);
        int g[8];
        for (int i = 0; i < 8; i++) g[i] = a.integer(4 + i);
        void* s = a.stream();
        run(decltype(&chipmunk_voxel_reorder){}, from, to, perm, inv, (int)src->size(0), g[0], g[1], g[2], g[3], g[4], g[5], g[6], g[7], (int)row,
            (int)(a.v[12] == Py_True), s);
    });
}

// cur, prev, k, idx, counts
PyObject* topk_cols(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return answer(kTopk, args, n, 5, [](Args& a, auto run) {
        auto rows = [&](int i) -> const at::Tensor* {   // dense rows that a leading dimension may space
            const at::Tensor* t = a.tensor(i);
            if (a.ok && (t->dim() != 2 || t->scalar_type() != at::kFloat || !t->is_cuda() || (t->size(1) > 1 && t->stride(1) != 1))) a.ok = false;
            return t;
        };
        const at::Tensor* cur = rows(0);
        const at::Tensor* prev = a.none(1) ? nullptr : rows(1);
        if (!a.ok || (prev && (prev->sizes() != cur->sizes() || prev->stride(0) != cur->stride(0))) || cur->size(0) > INT_MAX || cur->size(1) > INT_MAX) {
            a.ok = false;
            return;
        }
        const int k = a.integer(2);
        int32_t *idx = a.i32(3), *counts = a.i32(4);
        const int k_stride = a.size(3, -1, 0);
        void* s = a.stream();
        run(decltype(&chipmunk_topk_cols){}, (const float*)cur->data_ptr(), prev ? (const float*)prev->data_ptr() : nullptr, (int)cur->size(0), (int)cur->size(1),
            (int64_t)cur->stride(0), k, idx, counts, k_stride, s);
    });
}

// q, k, v, idx, counts, base, out, c, softmax_scale, o_scale
PyObject* attn_sparse_delta(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return answer(kAttnDelta, args, n, 10, [](Args& a, auto run) {
        const uint16_t *q = a.bf16(0), *k = a.bf16(1), *v = a.bf16(2);
        const int B = a.size(0, 4, 0), H = a.size(0, 4, 1), N = a.size(0, 4, 2), E = a.size(0, 4, 3);
        const int32_t *idx = a.i32(3), *counts = a.i32(4);
        const int k_stride = a.none(3) ? 0 : a.size(3, -1, 0);
        const uint16_t* base = a.bf16(5);
        uint16_t* out = a.bf16_out(6);
        const int c = a.integer(7);
        const float scale = a.real(8), o_scale = a.real(9);
        void* s = a.stream();
        run(decltype(&chipmunk_attn_sparse_delta){}, q, k, v, idx, counts, base, out, B, H, N, E, c, k_stride, scale, o_scale, s);
    });
}

// q, k, v, out, colsum, c, softmax_scale, ws
PyObject* attn_dense(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return answer(kAttnDense, args, n, 8, [](Args& a, auto run) {
        const uint16_t *q = a.bf16(0), *k = a.bf16(1), *v = a.bf16(2);
        const int B = a.size(0, 4, 0), H = a.size(0, 4, 1), N = a.size(0, 4, 2), E = a.size(0, 4, 3);
        uint16_t* out = a.bf16_out(3);
        float* colsum = a.f32(4);
        const int64_t ld = a.none(4) ? 0 : a.size(4, -1, 0);
        const int c = a.integer(5);
        const float scale = a.real(6);
        void* ws = a.data(7, at::kByte);
        const size_t bytes = a.elements(7);
        void* s = a.stream();
        run(decltype(&chipmunk_attn_dense){}, q, k, v, out, colsum, ld, B, H, N, E, c, scale, ws, bytes, s);
    });
}

// q, k, v, out, prev_m, prev_l, colsum, c, softmax_scale, new_m, new_l
PyObject* attn_dense_colsum_stale(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return answer(kAttnRefresh, args, n, 11, [](Args& a, auto run) {
        const uint16_t *q = a.bf16(0), *k = a.bf16(1), *v = a.bf16(2);
        const int B = a.size(0, 4, 0), H = a.size(0, 4, 1), N = a.size(0, 4, 2), E = a.size(0, 4, 3);
        uint16_t* out = a.bf16_out(3);
        const float *prev_m = a.f32(4), *prev_l = a.f32(5);
        float* colsum = a.f32(6);
        const int64_t ld = a.size(6, -1, 0);
        const int c = a.integer(7);
        const float scale = a.real(8);
        float *new_m = a.f32(9), *new_l = a.f32(10);
        void* s = a.stream();
        run(decltype(&chipmunk_attn_dense_colsum_stale){}, q, k, v, out, prev_m, prev_l, colsum, ld, new_m, new_l, B, H, N, E, c, scale, s);
    });
}

// x, w1, T, c, ws
PyObject* mlp_tile_mean_preact(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return answer(kScores, args, n, 5, [](Args& a, auto run) {
        const uint16_t *x = a.bf16(0), *w1 = a.bf16(1);
        const int B = a.size(0, 3, 0), N = a.size(0, 3, 1), D = a.size(0, 3, 2), F = a.rows(1);
        float* T = a.f32(2);
        const int c = a.integer(3);
        void* ws = a.data(4, at::kByte);
        const size_t bytes = a.elements(4);
        void* s = a.stream();
        run(decltype(&chipmunk_mlp_tile_mean_preact){}, x, w1, T, B, N, D, F, c, ws, bytes, s);
    });
}

// x, w1, b1, w2, idx, counts, a_cache, o_cache, c, act, ws
PyObject* mlp_sparse_delta(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return answer(kMlpDelta, args, n, 11, [](Args& a, auto run) {
        const uint16_t *x = a.bf16(0), *w1 = a.bf16(1), *b1 = a.bf16(2), *w2 = a.bf16(3);
        const int B = a.size(0, 3, 0), N = a.size(0, 3, 1), D = a.size(0, 3, 2), F = a.rows(1);
        const int32_t *idx = a.i32(4), *counts = a.i32(5);
        const int k_stride = a.size(4, -1, 0);
        uint16_t *a_cache = a.bf16_out(6), *o_cache = a.bf16_out(7);
        const int64_t a_ld = a.size(6, -1, 0);
        const int c = a.integer(8), act = a.integer(9);
        void* ws = a.data(10, at::kByte);
        const size_t bytes = a.elements(10);
        void* s = a.stream();
        run(decltype(&chipmunk_mlp_sparse_delta){}, x, w1, b1, w2, idx, counts, a_cache, a_ld, o_cache, B, N, D, F, c, k_stride, act, ws, bytes, s);
    });
}

// x, w1, b1, w2, b2, out, a_cache, c, act
PyObject* mlp_dense(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return answer(kMlpDense, args, n, 9, [](Args& a, auto run) {
        const uint16_t *x = a.bf16(0), *w1 = a.bf16(1), *b1 = a.bf16(2), *w2 = a.bf16(3), *b2 = a.bf16(4);
        const int B = a.size(0, 3, 0), N = a.size(0, 3, 1), D = a.size(0, 3, 2), F = a.rows(1);
        uint16_t *out = a.bf16_out(5), *a_cache = a.bf16_out(6);
        const int64_t a_ld = a.size(6, -1, 0);
        const int c = a.integer(7), act = a.integer(8);
        void* s = a.stream();
        run(decltype(&chipmunk_mlp_dense){}, x, w1, b1, w2, b2, out, a_cache, a_ld, B, N, D, F, c, act, s);
    });
}

// bind(addresses: dict of names, current_device, raw_stream)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 3 || !PyDict_Check(args[0])) {
        PyErr_SetString(PyExc_TypeError, "bind(addresses, current_device, raw_stream)");
        return nullptr;
    }
    for (Entry& e : entries) {
        PyObject* at = PyDict_GetItemString(args[0], e.name);
        e.at = at ? PyLong_AsVoidPtr(at) : nullptr;
        if (PyErr_Occurred()) return nullptr;
    }
    Py_INCREF(args[1]);
    Py_XSETREF(current_device, args[1]);
    Py_INCREF(args[2]);
    Py_XSETREF(raw_stream, args[2]);
    Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(bind), FAST(voxel_reorder), FAST(topk_cols), FAST(attn_sparse_delta), FAST(attn_dense),
                         FAST(attn_dense_colsum_stale), FAST(mlp_tile_mean_preact), FAST(mlp_sparse_delta), FAST(mlp_dense),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// The stamp names the torch, the Python and the header that this was compiled with.  It is looked for in the file before
// the file is loaded.
PyMODINIT_FUNC PyInit__native() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", CHIPMUNK_BINDING_STAMP) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
