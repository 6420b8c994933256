// The marshalling of the calls a training step is made of, in C++: what binding.py does for one of them in the interpreter
// (checks, output and workspace allocation, the call through ctypes) took 6 to 9 us of host time, about twice the launch itself.
//
// Every function returns the outputs, or the library's status as an int when that is not zero, or None when it does not take
// the call: anything unusual (other argument types, tensors that are no plain contiguous device tensors of the right element
// size, sizes that do not match) is left to the Python code, which decides and raises as before.  The library's functions come
// as addresses (init), so this object does not link against it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/positnn.h"

namespace {

enum Fn { GEMM, GEMM_WS, CONV_FWD, CONV_BWD_DATA, CONV_BWD_WEIGHT, CONV_WS, ROUND, CONVERT, RELU, RELU_BWD, MAXPOOL_FWD, MAXPOOL_BWD, AVGPOOL_FWD, AVGPOOL_BWD, COUNT };
void* g_fn[COUNT];

typedef pnn_conv2d_desc Desc;

// The formats, as init() got them from binding.py: bytes per element (0: no such format), type of a new tensor, types taken
struct Format {
    int size;
    at::ScalarType type;
    uint64_t fits;
};
constexpr long FORMATS = 128;
Format g_formats[FORMATS];

int elem_size(long f) { return f < 0 || f >= FORMATS ? 0 : g_formats[f].size; }

at::ScalarType dtype_of(long f) { return g_formats[f].type; }

bool dtype_fits(at::ScalarType t, long f) { return elem_size(f) && (g_formats[f].fits >> (int)t & 1u); }

// The tensor behind o if it is a plain contiguous device tensor of f's element size
const at::Tensor* tensor(PyObject* o, long f) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous() || !dtype_fits(t.scalar_type(), f)) return nullptr;
    return &t;
}

bool integer(PyObject* o, long* v) {
    if (!PyLong_Check(o)) return false;
    *v = PyLong_AsLong(o);
    if (*v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

at::Tensor empty(at::IntArrayRef shape, at::ScalarType t, const at::Tensor& like) { return at::empty(shape, at::TensorOptions().dtype(t).device(like.device())); }

// An output the caller gave, or null for a new one.  False: it does not fit.
bool given(PyObject* o, long f, const at::Tensor** out) {
    *out = o == Py_None ? nullptr : tensor(o, f);
    return o == Py_None || *out;
}

PyObject* none() { Py_RETURN_NONE; }

PyObject* result(int status, const at::Tensor& out) { return status ? PyLong_FromLong(status) : THPVariable_Wrap(out); }

PyObject* result(int status, const at::Tensor& a, const at::Tensor& b) {
    if (status) return PyLong_FromLong(status);
    PyObject* x = THPVariable_Wrap(a);
    PyObject* y = x ? THPVariable_Wrap(b) : nullptr;
    PyObject* r = y ? PyTuple_Pack(2, x, y) : nullptr;
    Py_XDECREF(x);
    Py_XDECREF(y);
    return r;
}

// Allocations and the call itself run without the interpreter's lock, as torch.empty and a call through ctypes do: other Python
// threads may run meanwhile, and the first allocation of a size can take long.  No Python object is touched inside.
class Unlocked {
    PyThreadState* state = PyEval_SaveThread();

public:
    Unlocked() = default;
    Unlocked(const Unlocked&) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};

template <class F, class... A>
int call(Fn which, A... args) { return reinterpret_cast<F>(g_fn[which])(args...); }

// Arguments: nints leading integers (the first the stream), then objects.
constexpr int MOST_INTS = 8;
struct Args {
    long i[MOST_INTS];
    void* stream;
    PyObject* const* o;
};

bool parse(PyObject* const* args, Py_ssize_t n, int nints, int nobjs, Args* a) {
    if (n != nints + nobjs) return false;
    for (int k = 0; k < nints; ++k)
        if (!integer(args[k], &a->i[k])) return false;
    a->stream = reinterpret_cast<void*>(a->i[0]);
    a->o = args + nints;
    return true;
}

// C++ exceptions (a functorch wrapper without storage, an allocation that fails) leave the call to the Python code, which meets
// the same and raises.
template <class B>
PyObject* guarded(const B& body) {
    try {
        return body();
    } catch (const std::exception&) {
        return none();
    }
}

typedef decltype(&posit_gemm) gemm_t;
typedef decltype(&posit_gemm_workspace) gemm_ws_t;
typedef decltype(&posit_conv2d_fwd) conv3_t;
typedef decltype(&posit_conv2d_bwd_data) conv_bd_t;
typedef decltype(&posit_conv2d_bwd_weight) conv_bw_t;
typedef decltype(&posit_conv2d_workspace) conv_ws_t;
typedef decltype(&posit_round) map_t;
typedef decltype(&posit_relu) relu_t;
typedef decltype(&posit_relu_bwd) relu_bwd_t;
typedef decltype(&posit_maxpool2d_fwd) maxpool_t;
typedef decltype(&posit_maxpool2d_bwd) maxpool_bwd_t;
typedef decltype(&posit_avgpool2d_fwd) avgpool_t;

// gemm(stream, fin, fout, trans_a, trans_b, A, B, bias, out)
PyObject* gemm(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a;
    if (!parse(args, n, 5, 4, &a)) return none();
    return guarded([&]() -> PyObject* {
        if (!elem_size(a.i[1]) || !elem_size(a.i[2])) return none();  // before they are narrowed
        const int fin = (int)a.i[1], fout = (int)a.i[2], ta = a.i[3] != 0, tb = a.i[4] != 0;
        const at::Tensor *A = tensor(a.o[0], fin), *B = tensor(a.o[1], fin), *bias = nullptr;
        if (!A || !B || A->dim() != 2 || B->dim() != 2) return none();
        const int64_t lda = A->size(1), ldb = B->size(1);
        const int64_t M = ta ? lda : A->size(0), K = ta ? A->size(0) : lda, N = tb ? B->size(0) : ldb;
        if (K != (tb ? ldb : B->size(0))) return none();
        if (a.o[2] != Py_None && (!(bias = tensor(a.o[2], fin)) || bias->numel() != N)) return none();
        const at::Tensor* to;
        if (!given(a.o[3], fout, &to) || (to && to->dim() != 2)) return none();
        at::Tensor out, ws;
        int status;
        {
            Unlocked here;
            out = to ? *to : empty({M, N}, dtype_of(fout), *A);
            const size_t bytes = reinterpret_cast<gemm_ws_t>(g_fn[GEMM_WS])(fin, fout, ta, tb, M, N, K);
            if (bytes) ws = empty({(int64_t)bytes}, at::kByte, *A);
            status = call<gemm_t>(GEMM, a.stream, fin, fout, ta, tb, M, N, K, (const void*)A->data_ptr(), lda, (const void*)B->data_ptr(), ldb,
                                  (const void*)(bias ? bias->data_ptr() : nullptr), (void*)out.data_ptr(), out.size(1), bytes ? (void*)ws.data_ptr() : nullptr, bytes);
        }
        return result(status, out);
    });
}

// conv(stream, which, fin, fout, desc, with_bias, first, second, bias, out, out_bias): first and second are x and w, dy and w, or dy and x
PyObject* conv(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a;
    if (!parse(args, n, 6, 5, &a)) return none();
    return guarded([&]() -> PyObject* {
        if (!elem_size(a.i[2]) || !elem_size(a.i[3])) return none();  // before they are narrowed
        const int which = (int)a.i[1], fin = (int)a.i[2], fout = (int)a.i[3];
        const Desc* d = reinterpret_cast<const Desc*>(a.i[4]);
        const bool with_bias = a.i[5] != 0;
        const at::Tensor *x = tensor(a.o[0], fin), *w = tensor(a.o[1], fin), *bias = nullptr;
        if (!x || !w) return none();
        if (a.o[2] != Py_None && !(bias = tensor(a.o[2], fin))) return none();
        const int64_t eh = d->H + 2 * d->pad_h - d->R, ew = d->W + 2 * d->pad_w - d->S;
        if (eh < 0 || ew < 0 || d->stride_h <= 0 || d->stride_w <= 0) return none();
        const at::Tensor *to, *to_bias = nullptr;
        if (!given(a.o[3], fout, &to) || (with_bias && !given(a.o[4], fout, &to_bias))) return none();
        at::Tensor out, db, ws;
        int status;
        {
            Unlocked here;
            const at::ScalarType t = dtype_of(fout);
            if (to) out = *to;
            else if (which == 0) out = empty({d->N, d->K, eh / d->stride_h + 1, ew / d->stride_w + 1}, t, *x);
            else if (which == 1) out = empty({d->N, d->C, d->H, d->W}, t, *x);
            else out = empty({d->K, d->C, d->R, d->S}, t, *x);
            if (with_bias) db = to_bias ? *to_bias : empty({d->K}, t, *x);
            const size_t bytes = reinterpret_cast<conv_ws_t>(g_fn[CONV_WS])(which, fin, fout, d);
            if (bytes) ws = empty({(int64_t)bytes}, at::kByte, *x);
            const void *xp = x->data_ptr(), *wp = w->data_ptr();
            void *op = out.data_ptr(), *sp = bytes ? ws.data_ptr() : nullptr;
            if (which == 0) status = call<conv3_t>(CONV_FWD, a.stream, fin, fout, d, xp, wp, (const void*)(bias ? bias->data_ptr() : nullptr), op, sp, bytes);
            else if (which == 1) status = call<conv_bd_t>(CONV_BWD_DATA, a.stream, fin, fout, d, xp, wp, op, sp, bytes);
            else status = call<conv_bw_t>(CONV_BWD_WEIGHT, a.stream, fin, fout, d, xp, wp, op, with_bias ? (void*)db.data_ptr() : nullptr, sp, bytes);
        }
        return with_bias ? result(status, out, db) : result(status, out);
    });
}

// round(stream, fdst, src, out), convert(stream, fsrc, fdst, src, out)
PyObject* map_elements(Fn fn, void* stream, long fsrc, long fdst, const at::Tensor* src, PyObject* dst) {
    const at::Tensor* to;
    if (!src || elem_size(fdst) == 0 || !given(dst, fdst, &to)) return none();
    at::Tensor out;
    int status;
    {
        Unlocked here;
        out = to ? *to : empty(src->sizes(), dtype_of(fdst), *src);
        status = call<map_t>(fn, stream, (int)fsrc, (int)fdst, src->numel(), (const void*)src->data_ptr(), (void*)out.data_ptr());
    }
    return result(status, out);
}

PyObject* round_to(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a;
    if (!parse(args, n, 2, 2, &a) || !THPVariable_CheckExact(a.o[0])) return none();
    return guarded([&]() -> PyObject* {
        const at::ScalarType t = THPVariable_Unpack(a.o[0]).scalar_type();
        if (t != at::kFloat && t != at::kDouble) return none();
        const long f = t == at::kFloat ? PNN_F32 : PNN_F64;
        return map_elements(ROUND, a.stream, f, a.i[1], tensor(a.o[0], f), a.o[1]);
    });
}

PyObject* convert(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a;
    if (!parse(args, n, 3, 2, &a)) return none();
    return guarded([&]() -> PyObject* { return map_elements(CONVERT, a.stream, a.i[1], a.i[2], tensor(a.o[0], a.i[1]), a.o[1]); });
}

// relu(stream, fmt, x, out)
PyObject* relu(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a;
    if (!parse(args, n, 2, 2, &a)) return none();
    return guarded([&]() -> PyObject* {
        const at::Tensor* x = tensor(a.o[0], a.i[1]);
        const at::Tensor* to;
        if (!x || !given(a.o[1], a.i[1], &to)) return none();
        at::Tensor out;
        int status;
        {
            Unlocked here;
            out = to ? *to : empty(x->sizes(), x->scalar_type(), *x);
            status = call<relu_t>(RELU, a.stream, (int)a.i[1], x->numel(), (const void*)x->data_ptr(), (void*)out.data_ptr());
        }
        return result(status, out);
    });
}

// relu_bwd(stream, fmt_y, fmt_d, y, dy, out)
PyObject* relu_bwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a;
    if (!parse(args, n, 3, 3, &a)) return none();
    return guarded([&]() -> PyObject* {
        const at::Tensor *y = tensor(a.o[0], a.i[1]), *dy = tensor(a.o[1], a.i[2]);
        const at::Tensor* to;
        if (!y || !dy || y->numel() != dy->numel() || !given(a.o[2], a.i[2], &to)) return none();
        at::Tensor out;
        int status;
        {
            Unlocked here;
            out = to ? *to : empty(dy->sizes(), dy->scalar_type(), *dy);
            status = call<relu_bwd_t>(RELU_BWD, a.stream, (int)a.i[1], (int)a.i[2], dy->numel(), (const void*)y->data_ptr(), (const void*)dy->data_ptr(),
                                      (void*)out.data_ptr());
        }
        return result(status, out);
    });
}

// Leading extent and shape of a pooled tensor: [..., H, W] with the last two divided or multiplied
struct Pool {
    int64_t planes, h, w;
    std::vector<int64_t> shape;
    bool of(const at::Tensor* t, long kh, long kw, bool up) {
        if (!t || t->dim() < 2 || kh <= 0 || kw <= 0) return false;
        h = t->size(-2);
        w = t->size(-1);
        if (h * w == 0) return false;
        planes = t->numel() / (h * w);
        shape = t->sizes().vec();
        shape[shape.size() - 2] = up ? h * kh : h / kh;
        shape[shape.size() - 1] = up ? w * kw : w / kw;
        return true;
    }
};

// maxpool_fwd(stream, fmt, kh, kw, x), maxpool_bwd(stream, fmt, kh, kw, dy, idx)
PyObject* maxpool_fwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a;
    if (!parse(args, n, 4, 1, &a)) return none();
    return guarded([&]() -> PyObject* {
        const at::Tensor* x = tensor(a.o[0], a.i[1]);
        Pool p;
        if (!p.of(x, a.i[2], a.i[3], false)) return none();
        at::Tensor y, idx;
        int status;
        {
            Unlocked here;
            y = empty(p.shape, x->scalar_type(), *x);
            idx = empty(p.shape, at::kByte, *x);
            status = call<maxpool_t>(MAXPOOL_FWD, a.stream, (int)a.i[1], p.planes, p.h, p.w, (int64_t)a.i[2], (int64_t)a.i[3], (const void*)x->data_ptr(),
                                     (void*)y.data_ptr(), (void*)idx.data_ptr());
        }
        return result(status, y, idx);
    });
}

PyObject* maxpool_bwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a;
    if (!parse(args, n, 4, 2, &a)) return none();
    return guarded([&]() -> PyObject* {
        const at::Tensor *dy = tensor(a.o[0], a.i[1]), *idx = tensor(a.o[1], PNN_POSIT8_0);
        Pool p;
        if (!idx || !p.of(dy, a.i[2], a.i[3], true)) return none();
        at::Tensor dx;
        int status;
        {
            Unlocked here;
            dx = empty(p.shape, dy->scalar_type(), *dy);
            status = call<maxpool_bwd_t>(MAXPOOL_BWD, a.stream, (int)a.i[1], p.planes, p.h * a.i[2], p.w * a.i[3], (int64_t)a.i[2], (int64_t)a.i[3],
                                     (const void*)dy->data_ptr(), (const void*)idx->data_ptr(), (void*)dx.data_ptr());
        }
        return result(status, dx);
    });
}

// avgpool(stream, backward, fin, fout, kh, kw, x)
PyObject* avgpool(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a;
    if (!parse(args, n, 6, 1, &a)) return none();
    return guarded([&]() -> PyObject* {
        const bool back = a.i[1] != 0;
        const long fin = a.i[2], fout = a.i[3], kh = a.i[4], kw = a.i[5];
        const at::Tensor* x = tensor(a.o[0], fin);
        Pool p;
        if (elem_size(fout) == 0 || !p.of(x, kh, kw, back)) return none();
        at::Tensor y;
        int status;
        {
            Unlocked here;
            y = empty(p.shape, dtype_of(fout), *x);
            status = call<avgpool_t>(back ? AVGPOOL_BWD : AVGPOOL_FWD, a.stream, (int)fin, (int)fout, p.planes, back ? p.h * kh : p.h, back ? p.w * kw : p.w, (int64_t)kh,
                                     (int64_t)kw, (const void*)x->data_ptr(), (void*)y.data_ptr());
        }
        return result(status, y);
    });
}

// init(formats, address ...): formats as rows (code, bytes, dtype, dtypes taken), the library's functions in the order of Fn
PyObject* init(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 1 + COUNT || !PyTuple_Check(args[0])) {
        PyErr_SetString(PyExc_TypeError, "the formats and one address per function");
        return nullptr;
    }
    for (Py_ssize_t k = 0; k < PyTuple_Size(args[0]); ++k) {
        long code;
        Format f;
        PyObject *type, *taken;
        if (!PyArg_ParseTuple(PyTuple_GetItem(args[0], k), "liO!O!", &code, &f.size, (PyTypeObject*)&THPDtypeType, &type, &PyTuple_Type, &taken)) return nullptr;
        f.type = reinterpret_cast<THPDtype*>(type)->scalar_type;
        f.fits = 0;
        for (Py_ssize_t i = 0; i < PyTuple_Size(taken); ++i) {
            PyObject* t = PyTuple_GetItem(taken, i);
            if (!THPDtype_Check(t) || (int)reinterpret_cast<THPDtype*>(t)->scalar_type >= 64) {
                PyErr_SetString(PyExc_TypeError, "a dtype");
                return nullptr;
            }
            f.fits |= (uint64_t)1 << (int)reinterpret_cast<THPDtype*>(t)->scalar_type;
        }
        if (code < 0 || code >= FORMATS) {
            PyErr_SetString(PyExc_ValueError, "format code");
            return nullptr;
        }
        g_formats[code] = f;
    }
    for (int k = 0; k < COUNT; ++k) {
        g_fn[k] = PyLong_AsVoidPtr(args[1 + k]);
        if (!g_fn[k]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
            return nullptr;
        }
    }
    Py_RETURN_NONE;
}

#define PNN_METHOD(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {PNN_METHOD("init", init), PNN_METHOD("gemm", gemm), PNN_METHOD("conv", conv), PNN_METHOD("round", round_to),
                         PNN_METHOD("convert", convert), PNN_METHOD("relu", relu), PNN_METHOD("relu_bwd", relu_bwd), PNN_METHOD("maxpool_fwd", maxpool_fwd),
                         PNN_METHOD("maxpool_bwd", maxpool_bwd), PNN_METHOD("avgpool", avgpool), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "positnn_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit_positnn_native() { return PyModule_Create(&module); }
