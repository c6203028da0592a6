// Argument marshalling of the Python binding in native code: turns tensors (anything with data_ptr(), stride(), shape and
// dtype), (address, leading dimension[, dtype]) sequences and None into the structures of the C ABI (include/tp_linear.h) and makes
// the call.  Nothing is computed, kept or checked here beyond that; the library answers for the arguments.
//
// Why: the smallest calls are shorter on the GPU than they were on the host.  A forward of 256 x 1024 x 4096 on a 2 x 2 grid spent
// 6.7 us in Python and ctypes before a call that takes 5.4 with its launch.
//
// The functions come from the loaded library by address (bind()), so this module links against nothing.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <new>
#include <vector>

#include "tp_linear.h"

namespace {

PyObject *s_data_ptr, *s_stride, *s_shape, *s_dtype, *s_numel, *s_element_size;      // interned names
PyObject *g_f32, *g_bf16;                                                            // torch.float32, torch.bfloat16

decltype(&tp_linear_fwd_ex) f_fwd;
decltype(&tp_linear_fwd_static) f_static;
decltype(&tp_linear_bwd_ex) f_bwd;
decltype(&tp_linear_bwd_partials_ex) f_partials;
decltype(&tp_bias_act) f_bias_act;
decltype(&tp_dgelu) f_dgelu;
decltype(&tp_bias_grad) f_bias_grad;

// Every helper returns false with a Python exception set.
struct Ref {                                       // an owned reference
    PyObject* p;
    explicit Ref(PyObject* q) : p(q) {}
    ~Ref() { Py_XDECREF(p); }
    Ref(const Ref&) = delete;
    Ref& operator=(const Ref&) = delete;
    explicit operator bool() const { return p != nullptr; }
};

bool to_i64(PyObject* o, int64_t* out) {           // int(o)
    if (PyLong_CheckExact(o)) {
        *out = (int64_t)PyLong_AsUnsignedLongLongMask(o);
        return !(*out == -1 && PyErr_Occurred());
    }
    Ref l(PyNumber_Long(o));
    if (!l) return false;
    *out = (int64_t)PyLong_AsUnsignedLongLongMask(l.p);
    return !(*out == -1 && PyErr_Occurred());
}
bool to_int(PyObject* o, int* out) {
    int64_t v;
    if (!to_i64(o, &v)) return false;
    *out = (int)v;
    return true;
}
bool call0(PyObject* o, PyObject* name, int64_t* out) {
    Ref r(PyObject_CallMethodNoArgs(o, name));
    return r && to_i64(r.p, out);
}
bool is_sequence(PyObject* o) { return PyTuple_Check(o) || PyList_Check(o); }
// a tensor has data_ptr; what has none is taken as a sequence
bool is_tensor(PyObject* o, bool* yes) {
    if (is_sequence(o)) { *yes = false; return true; }
    Ref a(PyObject_GetAttr(o, s_data_ptr));
    if (!a && !PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
    *yes = (bool)a;
    if (!a) PyErr_Clear();
    return true;
}
bool item(PyObject* o, Py_ssize_t i, int64_t* out) {
    Ref v(PySequence_GetItem(o, i));
    return v && to_i64(v.p, out);
}
// leading dimension: row stride of a 2-D tensor with unit column stride; a 1-D tensor is one row
bool tensor_ld(PyObject* t, int64_t* ld) {
    Ref st(PyObject_CallMethodNoArgs(t, s_stride));
    if (!st) return false;
    const Py_ssize_t n = PySequence_Size(st.p);
    if (n < 0) return false;
    if (n == 2) {
        int64_t cs;
        if (!item(st.p, 1, &cs)) return false;
        bool ok = cs == 1;
        if (!ok) {
            Ref sh(PyObject_GetAttr(t, s_shape));
            int64_t cols;
            if (!sh || !item(sh.p, 1, &cols)) return false;
            ok = cols <= 1;
        }
        if (ok) return item(st.p, 0, ld);
    } else if (n == 1) {
        Ref sh(PyObject_GetAttr(t, s_shape));
        return sh && item(sh.p, 0, ld);
    }
    PyErr_SetString(PyExc_ValueError, "blocks must be 2-D with unit column stride");
    return false;
}
bool to_cblk(PyObject* o, tp_cblk_t* b) {
    int64_t ptr = 0, ld = 0;
    if (o != Py_None) {
        bool tensor;
        if (!is_tensor(o, &tensor)) return false;
        if (tensor ? !(call0(o, s_data_ptr, &ptr) && tensor_ld(o, &ld)) : !(item(o, 0, &ptr) && item(o, 1, &ld))) return false;
    }
    b->ptr = reinterpret_cast<const void*>(ptr);
    b->ld = ld;
    return true;
}
bool to_oblk(PyObject* o, tp_oblk_t* b) {
    int64_t ptr = 0, ld = 0;
    int dtype = 0;
    if (o != Py_None) {
        bool tensor;
        if (!is_tensor(o, &tensor)) return false;
        if (tensor) {
            if (!call0(o, s_data_ptr, &ptr) || !tensor_ld(o, &ld)) return false;
            Ref dt(PyObject_GetAttr(o, s_dtype));
            if (!dt) return false;
            dtype = dt.p == g_f32 ? TP_F32 : dt.p == g_bf16 ? TP_BF16 : 99;       // 99: the library answers TP_ERR_DTYPE
        } else {
            int64_t d;
            if (!item(o, 0, &ptr) || !item(o, 1, &ld) || !item(o, 2, &d)) return false;
            dtype = (int)d;
        }
    }
    b->ptr = reinterpret_cast<void*>(ptr);
    b->ld = ld;
    b->dtype = dtype;
    return true;
}
bool to_ptr(PyObject* o, void** out) {             // None, a tensor or an address
    int64_t v = 0;
    if (o != Py_None) {
        if (PyLong_Check(o)) {
            if (!to_i64(o, &v)) return false;
        } else {
            bool tensor;
            if (!is_tensor(o, &tensor)) return false;
            if (tensor ? !call0(o, s_data_ptr, &v) : !to_i64(o, &v)) return false;
        }
    }
    *out = reinterpret_cast<void*>(v);
    return true;
}
struct Workspace { void* ptr; size_t bytes; };     // None, a tensor or (address, bytes)
bool to_ws(PyObject* o, Workspace* w) {
    int64_t ptr = 0, n = 0, each = 1;
    if (o != Py_None) {
        bool tensor;
        if (!is_tensor(o, &tensor)) return false;
        if (tensor ? !(call0(o, s_data_ptr, &ptr) && call0(o, s_numel, &n) && call0(o, s_element_size, &each)) : !(item(o, 0, &ptr) && item(o, 1, &n)))
            return false;
    }
    w->ptr = reinterpret_cast<void*>(ptr);
    w->bytes = (size_t)(n * each);
    return true;
}
bool to_dims(PyObject* o, tp_dims_t* d) {
    Ref s(PySequence_Fast(o, "dims must be (M, H, F)"));
    if (!s) return false;
    if (PySequence_Fast_GET_SIZE(s.p) != 3) {
        PyErr_SetString(PyExc_ValueError, "dims must be (M, H, F)");
        return false;
    }
    PyObject** it = PySequence_Fast_ITEMS(s.p);
    return to_i64(it[0], &d->M) && to_i64(it[1], &d->H) && to_i64(it[2], &d->F);
}
// A list of blocks, with empty ones up to TP_MAX_STEPS (the library reads no more); None: a null pointer.
template <class B, bool (*CONVERT)(PyObject*, B*)> struct Blocks {
    B fixed[TP_MAX_STEPS] = {};
    std::vector<B> more;
    const B* ptr = nullptr;
    bool fill(PyObject* o) {
        if (o == Py_None) return true;
        if (PyObject_Size(o) < 0) return false;    // (an iterator's blocks may be gone before the call)
        Ref s(PySequence_Fast(o, "blocks must be a sequence"));
        if (!s) return false;
        const Py_ssize_t n = PySequence_Fast_GET_SIZE(s.p);
        B* to = fixed;
        if (n > TP_MAX_STEPS) {
            try { more.resize((size_t)n); } catch (const std::bad_alloc&) { PyErr_NoMemory(); return false; }
            to = more.data();
        }
        for (Py_ssize_t i = 0; i < n; ++i)
            if (!CONVERT(PySequence_Fast_GET_ITEM(s.p, i), to + i)) return false;
        ptr = to;
        return true;
    }
};
using CBlocks = Blocks<tp_cblk_t, to_cblk>;
using OBlocks = Blocks<tp_oblk_t, to_oblk>;
struct MaybeBlock {                                // None: a null pointer
    tp_cblk_t b;
    const tp_cblk_t* ptr = nullptr;
    bool fill(PyObject* o) {
        if (o == Py_None) return true;
        if (!to_cblk(o, &b)) return false;
        ptr = &b;
        return true;
    }
};
template <class T> bool to_struct(PyObject* o, const T** out) {      // the address of a structure, 0 or None: none
    void* p;
    if (!to_ptr(o, &p)) return false;
    *out = static_cast<const T*>(p);
    return true;
}
bool count(Py_ssize_t have, Py_ssize_t want) {
    if (have == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, have);
    return false;
}
// The call itself runs without the interpreter lock: a launch waits when the stream's queue is full.
template <class F> PyObject* answer(F&& call) {
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// fwd(grid, dims, n_steps, x_blocks, w_blocks, bias, epi, y, preact, workspace, stream, opts)
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    const tp_grid_t* grid; const tp_plan_opts_t* opts;
    tp_dims_t dims; int steps, epi; CBlocks x, w; void *bias, *stream; tp_oblk_t y, pre; Workspace ws;
    if (!count(n, 12) || !to_struct(a[0], &grid) || !to_dims(a[1], &dims) || !to_int(a[2], &steps) || !x.fill(a[3]) || !w.fill(a[4]) ||
        !to_ptr(a[5], &bias) || !to_int(a[6], &epi) || !to_oblk(a[7], &y) || !to_oblk(a[8], &pre) || !to_ws(a[9], &ws) ||
        !to_ptr(a[10], &stream) || !to_struct(a[11], &opts))
        return nullptr;
    return answer([&] { return f_fwd(grid, &dims, steps, x.ptr, w.ptr, bias, epi, y, pre, ws.ptr, ws.bytes, stream, opts); });
}
// fwd_static(grid, dims, n_steps, x_blocks, w_blocks, bias, epi, y, preact, stream)
PyObject* fwd_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
    const tp_grid_t* grid;
    tp_dims_t dims; int steps, epi; CBlocks x, w; void *bias, *stream; tp_oblk_t y, pre;
    if (!count(n, 10) || !to_struct(a[0], &grid) || !to_dims(a[1], &dims) || !to_int(a[2], &steps) || !x.fill(a[3]) || !w.fill(a[4]) ||
        !to_ptr(a[5], &bias) || !to_int(a[6], &epi) || !to_oblk(a[7], &y) || !to_oblk(a[8], &pre) || !to_ptr(a[9], &stream))
        return nullptr;
    return answer([&] { return f_static(grid, &dims, steps, x.ptr, w.ptr, bias, epi, y, pre, stream); });
}
// bwd(grid, dims, n_dx, n_dw, dy_own, preact_own, da_row_blocks, w_blocks_dx, x_blocks_dw, da_col_blocks, own_slot_dx, own_slot_dw,
//     dgelu_preact, dx, dw, da_own_out, db, workspace, stream, opts)
PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    const tp_grid_t* grid; const tp_plan_opts_t* opts;
    tp_dims_t dims; int ndx, ndw, sdx, sdw; MaybeBlock dy, pre, dg; CBlocks rows, w, x, cols; tp_oblk_t dx, dw, da; void *db, *stream; Workspace ws;
    if (!count(n, 20) || !to_struct(a[0], &grid) || !to_dims(a[1], &dims) || !to_int(a[2], &ndx) || !to_int(a[3], &ndw) || !dy.fill(a[4]) ||
        !pre.fill(a[5]) || !rows.fill(a[6]) || !w.fill(a[7]) || !x.fill(a[8]) || !cols.fill(a[9]) || !to_int(a[10], &sdx) ||
        !to_int(a[11], &sdw) || !dg.fill(a[12]) || !to_oblk(a[13], &dx) || !to_oblk(a[14], &dw) || !to_oblk(a[15], &da) || !to_ptr(a[16], &db) ||
        !to_ws(a[17], &ws) || !to_ptr(a[18], &stream) || !to_struct(a[19], &opts))
        return nullptr;
    return answer([&] {
        return f_bwd(grid, &dims, ndx, ndw, dy.ptr, pre.ptr, rows.ptr, w.ptr, x.ptr, cols.ptr, sdx, sdw, dg.ptr, dx, dw, da, db, ws.ptr, ws.bytes,
                     stream, opts);
    });
}
// bwd_partials(grid, dims, n_dx, n_dw, da_own, w_blocks_dx, dx_partials, x_blocks_dw, dw_partials, workspace, stream, opts)
PyObject* bwd_partials(PyObject*, PyObject* const* a, Py_ssize_t n) {
    const tp_grid_t* grid; const tp_plan_opts_t* opts;
    tp_dims_t dims; int ndx, ndw; MaybeBlock da; CBlocks w, x; OBlocks dx, dw; void* stream; Workspace ws;
    if (!count(n, 12) || !to_struct(a[0], &grid) || !to_dims(a[1], &dims) || !to_int(a[2], &ndx) || !to_int(a[3], &ndw) || !da.fill(a[4]) ||
        !w.fill(a[5]) || !dx.fill(a[6]) || !x.fill(a[7]) || !dw.fill(a[8]) || !to_ws(a[9], &ws) || !to_ptr(a[10], &stream) ||
        !to_struct(a[11], &opts))
        return nullptr;
    return answer([&] { return f_partials(grid, &dims, ndx, ndw, da.ptr, w.ptr, dx.ptr, x.ptr, dw.ptr, ws.ptr, ws.bytes, stream, opts); });
}
// bias_act(c, bias, epi, y, preact, rows, cols, stream)
PyObject* bias_act(PyObject*, PyObject* const* a, Py_ssize_t n) {
    tp_cblk_t c; tp_oblk_t y, pre; void *bias, *stream; int epi; int64_t rows, cols;
    if (!count(n, 8) || !to_cblk(a[0], &c) || !to_ptr(a[1], &bias) || !to_int(a[2], &epi) || !to_oblk(a[3], &y) || !to_oblk(a[4], &pre) ||
        !to_i64(a[5], &rows) || !to_i64(a[6], &cols) || !to_ptr(a[7], &stream))
        return nullptr;
    return answer([&] { return f_bias_act(c.ptr, c.ld, bias, epi, y, pre, rows, cols, stream); });
}
// dgelu(dy, preact, da, rows, cols, stream)
PyObject* dgelu(PyObject*, PyObject* const* a, Py_ssize_t n) {
    tp_cblk_t dy, pre, da; void* stream; int64_t rows, cols;
    if (!count(n, 6) || !to_cblk(a[0], &dy) || !to_cblk(a[1], &pre) || !to_cblk(a[2], &da) || !to_i64(a[3], &rows) || !to_i64(a[4], &cols) ||
        !to_ptr(a[5], &stream))
        return nullptr;
    return answer([&] { return f_dgelu(dy.ptr, dy.ld, pre.ptr, pre.ld, const_cast<void*>(da.ptr), da.ld, rows, cols, stream); });
}
// bias_grad(da, db, rows, cols, workspace, stream)
PyObject* bias_grad(PyObject*, PyObject* const* a, Py_ssize_t n) {
    tp_cblk_t da; void *db, *stream; int64_t rows, cols; Workspace ws;
    if (!count(n, 6) || !to_cblk(a[0], &da) || !to_ptr(a[1], &db) || !to_i64(a[2], &rows) || !to_i64(a[3], &cols) || !to_ws(a[4], &ws) ||
        !to_ptr(a[5], &stream))
        return nullptr;
    return answer([&] { return f_bias_grad(da.ptr, da.ld, rows, cols, db, ws.ptr, ws.bytes, stream); });
}
// bind(addresses of the seven functions in the order above, torch.float32, torch.bfloat16)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    void* f[7];
    if (!count(n, 9)) return nullptr;
    for (int i = 0; i < 7; ++i)
        if (!to_ptr(a[i], &f[i])) return nullptr;
    f_fwd = reinterpret_cast<decltype(f_fwd)>(f[0]);
    f_static = reinterpret_cast<decltype(f_static)>(f[1]);
    f_bwd = reinterpret_cast<decltype(f_bwd)>(f[2]);
    f_partials = reinterpret_cast<decltype(f_partials)>(f[3]);
    f_bias_act = reinterpret_cast<decltype(f_bias_act)>(f[4]);
    f_dgelu = reinterpret_cast<decltype(f_dgelu)>(f[5]);
    f_bias_grad = reinterpret_cast<decltype(f_bias_grad)>(f[6]);
    Py_INCREF(a[7]); Py_XSETREF(g_f32, a[7]);
    Py_INCREF(a[8]); Py_XSETREF(g_bf16, a[8]);
    Py_RETURN_NONE;
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr
PyMethodDef methods[] = {{"fwd", FAST(fwd)}, {"fwd_static", FAST(fwd_static)}, {"bwd", FAST(bwd)}, {"bwd_partials", FAST(bwd_partials)},
                         {"bias_act", FAST(bias_act)}, {"dgelu", FAST(dgelu)}, {"bias_grad", FAST(bias_grad)}, {"bind", FAST(bind)},
                         {nullptr, nullptr, 0, nullptr}};
// (Set up in its exec slot: a second load of the file makes a module of its own.  A module set up in one go would fill the one that stands under
// this name in sys.modules, which may be another copy's.)
int exec(PyObject*) {
    struct { PyObject** to; const char* name; } names[] = {{&s_data_ptr, "data_ptr"}, {&s_stride, "stride"}, {&s_shape, "shape"},
                                                           {&s_dtype, "dtype"}, {&s_numel, "numel"}, {&s_element_size, "element_size"}};
    for (auto& x : names)
        if (!*x.to && !(*x.to = PyUnicode_InternFromString(x.name))) return -1;
    return 0;
}
PyModuleDef_Slot slots[] = {{Py_mod_exec, reinterpret_cast<void*>(exec)}, {0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tpcall", "argument marshalling of the libtplinear binding", 0, methods, slots, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tpcall(void) { return PyModuleDef_Init(&module); }
