// marshal.cpp -- the calls of binding.py that programs make step after step, marshalled in native code (a CPython extension; host
// only, no HIP call of its own).
//
// What bounds it: a small launch takes 2.0-2.5 us of the host, and ctypes and the checks of the tensors in Python cost as much again
// (1.0 us a call of seven arguments, 0.65 us a tensor).  Host time of a call, us, through ctypes -> here: a batched write of 2 plans
// 4.2 -> 3.0, of 64 4.3 -> 3.4; one plan's write 4.9 -> 3.1, read 4.7 -> 3.0; scores 6.1 -> 3.2; decode attention (two launches)
// 9.4 -> 6.0; srft_cache_append by way of lib() 0.3 less.
//
// A function here makes the call where everything is as binding.py wants it (plain tensors of the right type on the device, no
// stream named) and returns the status; it returns None where anything is not, before the call, and binding.py goes its own way,
// which raises what there is to raise.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>

#include "srft_kv.h"

namespace {

// ---- the C entry points, bound by binding.lib() when it loads the library; their types are the header's
struct {
    decltype(&srft_kv_quantize) quantize;
    decltype(&srft_kv_dequantize) dequantize;
    decltype(&srft_kv_quantize_batched) quantize_batched;
    decltype(&srft_kv_dequantize_batched) dequantize_batched;
    decltype(&srft_kv_scores) scores;
    decltype(&srft_kv_decode_attention) attention;
    decltype(&srft_kv_channel_absmax) absmax;
    decltype(&srft_cache_append) append;
    decltype(&srft_scores_workspace_bytes) scores_bytes;
    decltype(&srft_decode_attention_workspace_bytes) attention_bytes;
    decltype(&srft_plan_d) plan_d;
    bool bound;
} g;

// ---- arguments
template <class T>
bool handle_of(PyObject* o, T** p) {                         // a plan: the address as an int
    if (!PyLong_CheckExact(o)) return false;
    *p = (T*)PyLong_AsVoidPtr(o);
    if (*p || !PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}
// a plain contiguous tensor of this type on the device
const at::Tensor* tensor_of(PyObject* o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.scalar_type() == type && t.layout() == at::kStrided && t.unsafeGetTensorImpl()->has_storage() &&
                   t.is_contiguous()
               ? &t
               : nullptr;
}
PyTypeObject *cell_type, *array_type;                        // ctypes.c_void_p and ctypes.Array, with the entry points
bool address_of(PyObject* o, void** p) {                     // of a ctypes array or cell
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return false;
    }
    *p = b.buf;
    PyBuffer_Release(&b);
    return true;
}
uint8_t* codes_of(const at::Tensor* t) { return static_cast<uint8_t*>(t->data_ptr()); }
float* floats_of(const at::Tensor* t) { return static_cast<float*>(t->data_ptr()); }
void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Runs `body` (true: the call was made, its status in *rc), turning what it throws into "not made".
template <class F>
PyObject* made(F body) {
    int rc = 0;
    bool done = false;
    try {
        done = g.bound && body(&rc);
    } catch (...) {
    }
    if (done) return PyLong_FromLong(rc);
    Py_RETURN_NONE;
}
template <class F>
int without_gil(F call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return rc;
}
int64_t bytes_of(const at::Tensor& t) { return t.numel() * (int64_t)t.element_size(); }

// quantize(plan, x, codes, scales)
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return made([&](int* rc) {
        const srft_plan_t* plan;
        if (n != 4 || !handle_of(a[0], &plan)) return false;
        const at::Tensor *x = tensor_of(a[1], at::kHalf), *c = tensor_of(a[2], at::kByte), *s = tensor_of(a[3], at::kFloat);
        if (!x || !c || !s || x->dim() < 1) return false;
        void *const xp = x->data_ptr(), *const st = current_stream();
        uint8_t* const cp = codes_of(c);
        float* const sp = floats_of(s);
        const int64_t count = x->size(0);
        *rc = without_gil([&] { return g.quantize(plan, xp, count, cp, sp, st); });
        return true;
    });
}
// dequantize(plan, codes, scales, out)
PyObject* dequantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return made([&](int* rc) {
        const srft_plan_t* plan;
        if (n != 4 || !handle_of(a[0], &plan)) return false;
        const at::Tensor *c = tensor_of(a[1], at::kByte), *s = tensor_of(a[2], at::kFloat), *o = tensor_of(a[3], at::kHalf);
        if (!c || !s || !o || c->dim() < 1) return false;
        const uint8_t* const cp = codes_of(c);
        const float* const sp = floats_of(s);
        void *const op = o->data_ptr(), *const st = current_stream();
        const int64_t count = c->size(0);
        *rc = without_gil([&] { return g.dequantize(plan, cp, sp, count, op, st); });
        return true;
    });
}
// the arrays of a BatchTable
PyObject *s_plans, *s_big, *s_codes, *s_scales, *s_n_vec, *s_count;
PyObject* batched(PyObject* table, bool write) {
    PyObject* held[6] = {};                                  // (the arrays stay for the call, whatever happens to the table meanwhile)
    PyObject* const r = made([&](int* rc) {
        PyObject* const names[6] = {s_plans, s_big, s_codes, s_scales, s_n_vec, s_count};
        void* p[5];
        for (int i = 0; i < 6; ++i)
            if (!(held[i] = PyObject_GetAttr(table, names[i])) || (i < 5 && (!PyObject_TypeCheck(held[i], array_type) || !address_of(held[i], &p[i])))) {
                PyErr_Clear();
                return false;
            }
        int overflow;
        const long count = PyLong_CheckExact(held[5]) ? PyLong_AsLongAndOverflow(held[5], &overflow) : -1;
        if (count < 0 || count > INT32_MAX) return false;
        void* const st = current_stream();
        *rc = without_gil([&] {
            const auto plans = (const srft_plan_t* const*)p[0];
            const auto n_vec = (const int64_t*)p[4];
            return write ? g.quantize_batched(plans, (const void* const*)p[1], n_vec, (uint8_t* const*)p[2], (float* const*)p[3], (int)count, st)
                         : g.dequantize_batched(plans, (const uint8_t* const*)p[2], (const float* const*)p[3], n_vec, (void* const*)p[1], (int)count, st);
        });
        return true;
    });
    for (PyObject* o : held) Py_XDECREF(o);
    return r;
}
PyObject* quantize_batched(PyObject*, PyObject* table) { return batched(table, true); }
PyObject* dequantize_batched(PyObject*, PyObject* table) { return batched(table, false); }

// scores(plan, q, codes, scales, scores, workspace)
PyObject* scores(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return made([&](int* rc) {
        const srft_plan_t* plan;
        if (n != 6 || !handle_of(a[0], &plan) || !plan || !THPVariable_CheckExact(a[5])) return false;
        const at::Tensor *q = tensor_of(a[1], at::kHalf), *c = tensor_of(a[2], at::kByte), *s = tensor_of(a[3], at::kFloat),
                         *o = tensor_of(a[4], at::kFloat), *w = tensor_of(a[5], THPVariable_Unpack(a[5]).scalar_type());
        if (!q || !c || !s || !o || !w || q->dim() < 1 || c->dim() < 1 || o->dim() != 2 || o->size(0) != q->size(0) || o->size(1) != c->size(0) ||
            bytes_of(*w) < g.scores_bytes(plan))
            return false;
        const int64_t n_q = q->size(0), keys = c->size(0);
        const uint8_t* const cp = codes_of(c);
        const float* const sp = floats_of(s);
        float* const op = floats_of(o);
        void *const qp = q->data_ptr(), *const wp = w->data_ptr(), *const st = current_stream();
        if (n_q > INT32_MAX) return false;
        *rc = without_gil([&] { return g.scores(plan, qp, (int)n_q, cp, sp, keys, op, wp, st); });
        return true;
    });
}
// attention(plan_k, plan_v, q, k_codes, k_scales, v_codes, v_scales, softmax_scale, out, workspace)
PyObject* attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return made([&](int* rc) {
        const srft_plan_t *pk, *pv;
        if (n != 10 || !handle_of(a[0], &pk) || !handle_of(a[1], &pv) || !pk || !pv || !PyFloat_CheckExact(a[7]) || !THPVariable_CheckExact(a[9])) return false;
        const at::Tensor *q = tensor_of(a[2], at::kHalf), *kc = tensor_of(a[3], at::kByte), *ks = tensor_of(a[4], at::kFloat), *vc = tensor_of(a[5], at::kByte),
                         *vs = tensor_of(a[6], at::kFloat), *o = tensor_of(a[8], at::kFloat), *w = tensor_of(a[9], THPVariable_Unpack(a[9]).scalar_type());
        if (!q || !kc || !ks || !vc || !vs || !o || !w || q->dim() < 1 || kc->dim() < 1 || vc->dim() < 1 || vc->size(0) != kc->size(0)) return false;
        const int64_t n_q = q->size(0), keys = kc->size(0);
        if (n_q > INT32_MAX || bytes_of(*w) < g.attention_bytes(pk, pv, (int)n_q, keys)) return false;
        const float scale = (float)PyFloat_AS_DOUBLE(a[7]);
        const uint8_t *const kcp = codes_of(kc), *const vcp = codes_of(vc);
        const float *const ksp = floats_of(ks), *const vsp = floats_of(vs);
        float* const op = floats_of(o);
        void *const qp = q->data_ptr(), *const wp = w->data_ptr(), *const st = current_stream();
        *rc = without_gil([&] { return g.attention(pk, pv, qp, (int)n_q, kcp, ksp, vcp, vsp, keys, scale, op, wp, st); });
        return true;
    });
}
// absmax(plan, x, amax)
PyObject* absmax(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return made([&](int* rc) {
        const srft_plan_t* plan;
        if (n != 3 || !handle_of(a[0], &plan) || !plan) return false;
        const at::Tensor *x = tensor_of(a[1], at::kHalf), *m = tensor_of(a[2], at::kFloat);
        if (!x || !m || x->dim() < 1 || m->numel() != g.plan_d(plan)) return false;
        const int64_t count = x->size(0);
        void *const xp = x->data_ptr(), *const st = current_stream();
        float* const mp = floats_of(m);
        *rc = without_gil([&] { return g.absmax(plan, xp, count, mp, st); });
        return true;
    });
}

// ---- lib().srft_cache_append, a ctypes function of a type of its own whose calls come here first: those with other arguments than
// None, ints, c_void_p and arrays of them go on to ctypes.  (As the type's slot: by way of a __call__ in Python's sight a call took 0.03 us
// more.)
bool pointer_of(PyObject* o, void** p) {
    if (o == Py_None) {
        *p = nullptr;
        return true;
    }
    if (handle_of(o, p)) return true;
    const bool cell = Py_TYPE(o) == cell_type;
    if (!cell && !PyObject_TypeCheck(o, array_type)) return false;
    void* at;
    if (!address_of(o, &at)) return false;
    if (cell) std::memcpy(p, at, sizeof(*p));
    else *p = at;
    return true;
}
PyObject* append_call(PyObject* self, PyObject* args, PyObject* names) {
    void *cache, *fresh, *st;
    if (PyTuple_GET_SIZE(args) == 4 && !names && g.bound) {
        PyObject* const* a = &PyTuple_GET_ITEM(args, 0);
        if (pointer_of(a[0], &cache) && pointer_of(a[1], &fresh) && PyLong_CheckExact(a[2]) && pointer_of(a[3], &st)) {
            int overflow;
            const long t = PyLong_AsLongAndOverflow(a[2], &overflow);
            if (!overflow && t == (int)t)
                return PyLong_FromLong(without_gil([&] { return g.append((srft_cache_t*)cache, (const void* const*)fresh, (int)t, st); }));
        }
    }
    PyTypeObject* base = Py_TYPE(self);
    while (base->tp_call == append_call) base = base->tp_base;
    return base->tp_call(self, args, names);
}
// append(type, native): calls of the type's objects come here, or go to ctypes (again)
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 2 || !PyType_Check(a[0]) || !(((PyTypeObject*)a[0])->tp_flags & Py_TPFLAGS_HEAPTYPE)) {
        PyErr_SetString(PyExc_TypeError, "append(type, native)");
        return nullptr;
    }
    PyTypeObject* const type = (PyTypeObject*)a[0];
    type->tp_call = a[1] == Py_True ? append_call : type->tp_base->tp_call;
    PyType_Modified(type);
    Py_RETURN_NONE;
}

// bind(addresses, c_void_p, Array): of the entry points, in the order of the struct above.  True: they are the ones called here; False: those
// of another library are, which came first.
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    constexpr int kCount = 11;
    void* p[kCount];
    if (n != kCount + 2 || !PyType_Check(a[kCount]) || !PyType_Check(a[kCount + 1])) {
        PyErr_SetString(PyExc_TypeError, "bind takes the addresses of 11 entry points, c_void_p and Array");
        return nullptr;
    }
    for (int i = 0; i < kCount; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no entry point");
            return nullptr;
        }
    }
    if (g.bound) return PyBool_FromLong(std::memcmp(&g, p, sizeof(p)) == 0);
    cell_type = (PyTypeObject*)Py_NewRef(a[kCount]);
    array_type = (PyTypeObject*)Py_NewRef(a[kCount + 1]);
    std::memcpy(&g, p, sizeof(p));
    g.bound = true;
    Py_RETURN_TRUE;
}
static_assert(offsetof(decltype(g), bound) == 11 * sizeof(void*), "bind fills the pointers in order");

#define FAST(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(quantize), FAST(dequantize), FAST(scores), FAST(attention), FAST(absmax), FAST(append), FAST(bind),
                         {"quantize_batched", quantize_batched, METH_O, nullptr},
                         {"dequantize_batched", dequantize_batched, METH_O, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
    struct { PyObject** at; const char* name; } const names[] = {{&s_plans, "plans"}, {&s_big, "big"}, {&s_codes, "codes"}, {&s_scales, "scales"}, {&s_n_vec, "n_vec"}, {&s_count, "count"}};
    for (const auto& e : names)
        if (!(*e.at = PyUnicode_InternFromString(e.name))) return nullptr;
    return PyModule_Create(&module);
}
