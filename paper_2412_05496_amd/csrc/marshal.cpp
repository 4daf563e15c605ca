// The argument marshalling of binding.py for the calls of a training step and a decoding loop, in C++: a small call is bound
// by its host side, of which building the C structures from Python took 3 to 5 us (forward over 256 tokens 9.2 -> 4.3 us
// of host time, a decode with two launches 10.4 -> 7.3, with one 7.4 -> 4.2).
//
// Every function returns the status of the C entry point, or None where anything about the arguments is not plain
// (a type, layout, shape or range that the Python side refuses or converts, a subclass, a tensor without storage):
// binding.py then takes its own path, which decides what happens.  Nothing has been launched in that case.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/autograd/python_variable.h>

#include "flexattn.h"

namespace {

struct NotPlain {};
void require(bool ok) {
    if (!ok) throw NotPlain{};
}

PyTypeObject* g_params_type = nullptr;      // binding.ModParams, binding.BlockMask
PyTypeObject* g_blockmask_type = nullptr;
decltype(&flexattn_forward) g_forward = nullptr;
decltype(&flexattn_paged_forward) g_paged_forward = nullptr;
decltype(&flexattn_backward) g_backward = nullptr;
decltype(&flexattn_backward_stored) g_backward_stored = nullptr;
decltype(&flexattn_blockmask_build) g_blockmask_build = nullptr;
decltype(&flexattn_paged_convert_blockmask) g_convert = nullptr;
decltype(&flexattn_paged_decode) g_decode = nullptr;

// A reference that is given back.
struct Ref {
    PyObject* o;
    explicit Ref(PyObject* o_) : o(o_) { require(o != nullptr); }
    Ref(const Ref&) = delete;
    ~Ref() { Py_DECREF(o); }
};

int64_t integer(PyObject* o) {
    require(PyLong_CheckExact(o));
    int overflow = 0;
    const int64_t v = PyLong_AsLongLongAndOverflow(o, &overflow);
    require(!overflow);
    return v;
}
int32_t int32(int64_t v) {
    require(v >= INT32_MIN && v <= INT32_MAX);
    return (int32_t)v;
}
uint32_t uint32(PyObject* o) {
    const int64_t v = integer(o);
    require(v >= 0 && v <= UINT32_MAX);
    return (uint32_t)v;
}
float real(PyObject* o) {
    if (PyLong_CheckExact(o)) return (float)integer(o);
    require(PyFloat_CheckExact(o));
    return (float)PyFloat_AS_DOUBLE(o);
}
const at::Tensor& tensor(PyObject* o) {
    require(THPVariable_CheckExact(o));
    return THPVariable_Unpack(o);
}
void* data(PyObject* o) { return tensor(o).data_ptr(); }
void* data_or_null(PyObject* o) { return o == Py_None ? nullptr : data(o); }

// binding._tensor
flexattn_tensor rows(PyObject* o) {
    const at::Tensor& t = tensor(o);
    require(t.is_cuda() && t.scalar_type() == at::kBFloat16 && t.dim() == 4);
    const auto st = t.strides();
    require(st[3] == 1);
    return {t.data_ptr(), st[0], st[1], st[2]};
}
// binding._dims
flexattn_dims dims(PyObject* q_, PyObject* k_) {
    const at::Tensor &q = tensor(q_), &k = tensor(k_);
    require(q.dim() == 4 && k.dim() == 4);
    return {int32(q.size(0)), int32(q.size(1)), int32(k.size(1)), int32(q.size(2)), int32(k.size(2)), int32(q.size(3))};
}
float* lse(PyObject* o, PyObject* q_) {
    const at::Tensor &t = tensor(o), &q = tensor(q_);
    require(t.scalar_type() == at::kFloat && t.is_contiguous() && t.sizes() == q.sizes().slice(0, 3));
    return (float*)t.data_ptr();
}

PyObject* interned(const char* s) { return PyUnicode_InternFromString(s); }
#define ATTR(obj, name) ([](PyObject* o_) { static PyObject* const n_ = interned(name); return PyObject_GetAttr(o_, n_); }(obj))

int32_t int_attr(PyObject* value) {
    const Ref v(value);
    return int32(integer(v.o));
}
void* ptr_attr(PyObject* value, bool nullable = false) {
    const Ref v(value);
    return nullable ? data_or_null(v.o) : data(v.o);
}
void* array_attr(PyObject* value, at::ScalarType type, int64_t* last = nullptr) {
    const Ref v(value);
    if (v.o == Py_None) return nullptr;
    const at::Tensor& t = tensor(v.o);
    require(t.scalar_type() == type && t.is_cuda() && t.is_contiguous());
    if (last) {
        require(t.dim() > 0);
        *last = t.size(-1);
    }
    return t.data_ptr();
}
// binding.ModParams._c
flexattn_mod_params mod_params(PyObject* p) {
    require(Py_TYPE(p) == g_params_type);
    flexattn_mod_params c = {};
    c.window = int_attr(ATTR(p, "window"));
    c.prefix_len = int_attr(ATTR(p, "prefix_len"));
    {
        const Ref v(ATTR(p, "softcap"));
        c.softcap = real(v.o);
    }
    {
        const Ref v(ATTR(p, "doc_ids"));
        if (v.o != Py_None) {
            const at::Tensor& t = tensor(v.o);
            require(t.scalar_type() == at::kInt && t.is_cuda() && t.dim() > 0 && t.stride(-1) == 1);
            c.doc_ids = (const int32_t*)t.data_ptr();
            c.doc_stride_b = t.dim() == 2 && t.size(0) > 1 ? t.stride(0) : 0;
        }
    }
    c.alibi_bias = (const float*)array_attr(ATTR(p, "alibi_bias"), at::kFloat);
    int64_t rel_len = 0;
    c.rel_bias = (const float*)array_attr(ATTR(p, "rel_bias"), at::kFloat, &rel_len);
    c.rel_len = int32(rel_len);
    c.ctx_lens = (const int32_t*)array_attr(ATTR(p, "ctx_lens"), at::kInt);
    c.q_offsets = (const int32_t*)array_attr(ATTR(p, "q_offsets"), at::kInt);
    c.na_width = int_attr(ATTR(p, "na_width"));
    c.na_height = int_attr(ATTR(p, "na_height"));
    c.na_kernel = int_attr(ATTR(p, "na_kernel"));
    c.na_layout = int_attr(ATTR(p, "na_layout"));
    c.na_tile = int_attr(ATTR(p, "na_tile"));
    return c;
}
// binding.BlockMask._c
flexattn_blockmask blockmask(PyObject* b) {
    require(Py_TYPE(b) == g_blockmask_type);
    flexattn_blockmask c = {};
    c.Bm = int_attr(ATTR(b, "Bm"));
    c.Hm = int_attr(ATTR(b, "Hm"));
    c.q_len = int_attr(ATTR(b, "q_len"));
    c.kv_len = int_attr(ATTR(b, "kv_len"));
    c.Bq = int_attr(ATTR(b, "Bq"));
    c.Bk = int_attr(ATTR(b, "Bk"));
    c.kv_num_blocks = (int32_t*)ptr_attr(ATTR(b, "kv_num_blocks"));
    c.kv_indices = (int32_t*)ptr_attr(ATTR(b, "kv_indices"));
    c.full_kv_num_blocks = (int32_t*)ptr_attr(ATTR(b, "full_kv_num_blocks"));
    c.full_kv_indices = (int32_t*)ptr_attr(ATTR(b, "full_kv_indices"));
    c.q_num_blocks = (int32_t*)ptr_attr(ATTR(b, "q_num_blocks"));
    c.q_indices = (int32_t*)ptr_attr(ATTR(b, "q_indices"));
    c.full_q_num_blocks = (int32_t*)ptr_attr(ATTR(b, "full_q_num_blocks"));
    c.full_q_indices = (int32_t*)ptr_attr(ATTR(b, "full_q_indices"));
    c.kv_order = (int32_t*)ptr_attr(ATTR(b, "kv_order"), true);
    c.q_order = (int32_t*)ptr_attr(ATTR(b, "q_order"), true);
    return c;
}
// what binding._stream, which is passed as a function, returns: asked for last, when all else is plain
void* stream(PyObject* f) {
    const Ref v(PyObject_CallNoArgs(f));
    require(PyLong_CheckExact(v.o));
    return PyLong_AsVoidPtr(v.o);
}

// call() prepares the arguments and returns the launch, which runs without the interpreter lock
template <typename F>
PyObject* run(Py_ssize_t n, Py_ssize_t want, F&& call) {
    try {
        require(n == want && !at::impl::torch_function_mode_enabled());
        auto launch = call();
        int status;
        Py_BEGIN_ALLOW_THREADS;
        status = launch();
        Py_END_ALLOW_THREADS;
        return PyLong_FromLong(status);
    } catch (...) {             // (of torch as well: a tensor without storage)
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// Q, K, V, score_id, mask_id, params, bm, scale, O, LSE, stream
PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return run(n, 11, [&] {
        return [d = dims(a[0], a[1]), q = rows(a[0]), k = rows(a[1]), v = rows(a[2]), score = uint32(a[3]), mask = uint32(a[4]),
                p = mod_params(a[5]), bm = blockmask(a[6]), scale = real(a[7]), o = rows(a[8]), l = lse(a[9], a[0]), st = stream(a[10])] {
            return g_forward(&d, &q, &k, &v, score, mask, &p, &bm, scale, &o, l, st);
        };
    });
}
// Q, K_pool, V_pool, score_id, mask_id, params, bm, phys_kv_indices, phys_full_kv_indices, scale, O, LSE, stream
PyObject* paged_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return run(n, 13, [&] {
        const at::Tensor &q = tensor(a[0]), &kp = tensor(a[1]), &vp = tensor(a[2]);
        require(q.dim() == 4 && kp.dim() == 4 && kp.is_contiguous() && vp.is_contiguous() && kp.sizes() == vp.sizes());
        const Ref kv(ATTR(a[6], "kv_indices")), full(ATTR(a[6], "full_kv_indices"));
        PyObject* const logical[2] = {kv.o, full.o};
        for (int i = 0; i < 2; ++i) {
            const at::Tensor& phys = tensor(a[7 + i]);
            require(phys.scalar_type() == at::kInt && phys.is_contiguous() && phys.sizes() == tensor(logical[i]).sizes());
        }
        const flexattn_blockmask bm = blockmask(a[6]);
        const flexattn_dims d = {int32(q.size(0)), int32(q.size(1)), int32(kp.size(1)), int32(q.size(2)), bm.kv_len, int32(kp.size(3))};
        return [d, bm, tq = rows(a[0]), k = kp.data_ptr(), v = vp.data_ptr(), page = int32(kp.size(2)), pool = int32(kp.size(0)),
                score = uint32(a[3]), mask = uint32(a[4]), p = mod_params(a[5]), phys = (const int32_t*)data(a[7]),
                phys_full = (const int32_t*)data(a[8]), scale = real(a[9]), o = rows(a[10]), l = lse(a[11], a[0]), st = stream(a[12])] {
            return g_paged_forward(&d, &tq, k, v, page, pool, score, mask, &p, &bm, phys, phys_full, scale, &o, l, st);
        };
    });
}
// Q, K, V, O, dO, LSE, score_id, mask_id, params, bm, scale, dQ, dK, dV, ws, stream
PyObject* backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return run(n, 16, [&] {
        return [d = dims(a[0], a[1]), q = rows(a[0]), k = rows(a[1]), v = rows(a[2]), o = rows(a[3]), dout = rows(a[4]), l = (const float*)data(a[5]),
                score = uint32(a[6]), mask = uint32(a[7]), p = mod_params(a[8]), bm = blockmask(a[9]), scale = real(a[10]), dq = rows(a[11]),
                dk = rows(a[12]), dv = rows(a[13]), ws = data(a[14]), bytes = (size_t)tensor(a[14]).numel(), st = stream(a[15])] {
            return g_backward(&d, &q, &k, &v, &o, &dout, l, score, mask, &p, &bm, scale, &dq, &dk, &dv, ws, bytes, st);
        };
    });
}
// Q, K, V, O, dO, LSE, score_id, mask_id, params, bm, scale, dQ, dK, dV, n_blocks, ws, stages, stream
PyObject* backward_stored(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return run(n, 18, [&] {
        return [d = dims(a[0], a[1]), q = rows(a[0]), k = rows(a[1]), v = rows(a[2]), o = rows(a[3]), dout = rows(a[4]), l = (const float*)data(a[5]),
                score = uint32(a[6]), mask = uint32(a[7]), p = mod_params(a[8]), bm = blockmask(a[9]), scale = real(a[10]), dq = rows(a[11]),
                dk = rows(a[12]), dv = rows(a[13]), blocks = integer(a[14]), ws = data(a[15]), bytes = (size_t)tensor(a[15]).numel(),
                stages = uint32(a[16]), st = stream(a[17])] {
            return g_backward_stored(&d, &q, &k, &v, &o, &dout, l, score, mask, &p, &bm, scale, &dq, &dk, &dv, blocks, ws, bytes, st, stages);
        };
    });
}
// mask_id, params, bm, ws, stream
PyObject* blockmask_build(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return run(n, 5, [&] {
        return [mask = uint32(a[0]), p = mod_params(a[1]), bm = blockmask(a[2]), stats = (int64_t*)ptr_attr(ATTR(a[2], "stats"), true),
                ws = data(a[3]), bytes = (size_t)tensor(a[3]).numel(), st = stream(a[4])] {
            return g_blockmask_build(mask, &p, &bm, stats, ws, bytes, st);
        };
    });
}
// num_blocks, indices, page_table, phys_indices, phys2log, stream
PyObject* convert(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return run(n, 6, [&] {
        const at::Tensor &idx = tensor(a[1]), &table = tensor(a[2]);
        require(idx.dim() == 4 && table.dim() > 0);
        const int32_t pool = a[4] == Py_None ? INT32_MAX : int32(tensor(a[4]).numel());
        return [num = (const int32_t*)data(a[0]), in = (const int32_t*)idx.data_ptr(), Bm = int32(idx.size(0)), Hm = int32(idx.size(1)),
                NR = int32(idx.size(2)), NC = int32(idx.size(3)), t = (const int32_t*)table.data_ptr(), ts = table.stride(0),
                out = (int32_t*)data(a[3]), back = (int32_t*)data_or_null(a[4]), pool, st = stream(a[5])] {
            return g_convert(num, in, Bm, Hm, NR, NC, t, ts, out, back, pool, st);
        };
    });
}
// Q, K_pool, V_pool, page_table, ctx_lens, score_id, mask_id, params, scale, O, LSE, ws, stream
PyObject* paged_decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return run(n, 13, [&] {
        const at::Tensor &q = tensor(a[0]), &kp = tensor(a[1]), &vp = tensor(a[2]), &table = tensor(a[3]), &o = tensor(a[9]);
        require(kp.is_contiguous() && vp.is_contiguous() && o.is_contiguous() && q.dim() >= 2 && kp.dim() == 4 && table.dim() == 2);
        require(q.stride(-1) == 1 && q.stride(1) == q.size(-1));
        const flexattn_decode_dims d = {int32(q.size(0)), int32(q.size(1)), int32(kp.size(1)), int32(q.size(-1)), int32(kp.size(2)),
                                        int32(table.size(1)), int32(kp.size(0))};
        return [d, qp = q.data_ptr(), qs = q.stride(0), k = kp.data_ptr(), v = vp.data_ptr(), t = (const int32_t*)table.data_ptr(), ts = table.stride(0),
                ctx = (const int32_t*)data(a[4]), score = uint32(a[5]), mask = uint32(a[6]), p = mod_params(a[7]), scale = real(a[8]),
                op = o.data_ptr(), l = (float*)data_or_null(a[10]), ws = data(a[11]), bytes = (size_t)tensor(a[11]).numel(), st = stream(a[12])] {
            return g_decode(&d, qp, qs, k, v, t, ts, ctx, score, mask, &p, scale, op, l, ws, bytes, st);
        };
    });
}

// ModParams, BlockMask, and the addresses of the entry points in the order below
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 9 || !PyType_Check(a[0]) || !PyType_Check(a[1])) {
        PyErr_SetString(PyExc_TypeError, "setup(ModParams, BlockMask, seven addresses)");
        return nullptr;
    }
    void* at[7];
    for (int i = 0; i < 7; ++i) {
        at[i] = PyLong_AsVoidPtr(a[2 + i]);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_INCREF(a[0]);
    Py_INCREF(a[1]);
    g_params_type = (PyTypeObject*)a[0];
    g_blockmask_type = (PyTypeObject*)a[1];
    g_forward = (decltype(g_forward))at[0];
    g_paged_forward = (decltype(g_paged_forward))at[1];
    g_backward = (decltype(g_backward))at[2];
    g_backward_stored = (decltype(g_backward_stored))at[3];
    g_blockmask_build = (decltype(g_blockmask_build))at[4];
    g_convert = (decltype(g_convert))at[5];
    g_decode = (decltype(g_decode))at[6];
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {METHOD(forward), METHOD(paged_forward), METHOD(backward), METHOD(backward_stored), METHOD(blockmask_build),
                          METHOD(convert), METHOD(paged_decode), METHOD(setup), {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&kModule); }
