// The marshalling of the layer calls, natively.  A call through ctypes with some twenty arguments, each looked up on a
// tensor from Python, takes 10 us, more than a small layer takes on the GPU; here it takes under 1 us (16 tokens, 512 x
// 512, 32 outliers, one call after another: 14.4 -> 8.2 us).  Only the ordinary call is served: plain device tensors of
// the documented types and strides, the output and the workspace given.  Everything else -- missing buffers, other types
// or strides, tensor subclasses, transformed tensors -- is answered with None, and the Python binding (api.py) does what
// it does without this file, errors included.
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>

#include <climits>
#include <cstdint>
#include <type_traits>

namespace {

// addresses of the library's entry points (bind)
struct Entry {
    int (*linear)(const void*, int, int, int, const int32_t*, int, int, const void*, int, const void*, const float*, const void*,
                  int, const void*, int, void*, int, void*, size_t, void*);
    int (*linear_w4a8)(const void*, int, int, int, const int32_t*, int, const void*, int, const void*, const float*, const void*,
                       int, const void*, int, void*, int, void*, size_t, void*);
    int (*linear_fp6)(const void*, int, int, int, const int32_t*, int, const void*, const void*, const float*, const void*, int,
                      const void*, int, void*, int, void*, size_t, void*);
    int (*linear_sp24)(const void*, int, int, int, const int32_t*, int, const void*, const void*, const float*, const void*, int,
                       const void*, int, void*, int, void*, size_t, void*);
    int (*quantize)(const void*, int, int, int, const int32_t*, int, int, void*, int, float*, float*, void*, int, void*, size_t,
                    void*);
    int (*gemm_dequant)(const void*, int, const float*, const float*, const void*, int, int, int, int, int, const void*, int,
                        const void*, const float*, const void*, int, const void*, int, void*, int, const void*, size_t, void*);
} entry;

const c10::DispatchKeySet kWrapped({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::Batched,
                                    c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                    c10::DispatchKey::ZeroTensor});

// an argument: a plain device tensor, or None (t == nullptr); `ok` is false for anything else
struct Arg {
    const at::Tensor* t = nullptr;
    bool ok = true;
    explicit Arg(PyObject* o) {
        if (o == Py_None) return;
        ok = THPVariable_CheckExact(o);
        if (!ok) return;
        t = &THPVariable_Unpack(o);
        ok = t->defined() && t->is_cuda() && t->layout() == c10::kStrided && t->has_storage() && !t->key_set().has_any(kWrapped);
    }
    void* ptr() const { return t ? t->data_ptr() : nullptr; }
    // a matrix with contiguous rows whose sizes are ints
    bool matrix() const {
        return t && t->dim() == 2 && t->stride(1) == 1 && t->size(0) <= INT_MAX && t->size(1) <= INT_MAX && t->stride(0) >= 0 &&
               t->stride(0) <= INT_MAX;
    }
    bool matrix(c10::ScalarType type) const { return matrix() && t->scalar_type() == type; }
    // consecutive elements of a type
    bool vector(c10::ScalarType type) const { return t && t->scalar_type() == type && t->is_contiguous(); }
    bool vector_or_none(c10::ScalarType type) const { return !t || vector(type); }
    bool buffer_or_none() const { return !t || t->is_contiguous(); }
    int rows() const { return (int)t->size(0); }
    int cols() const { return (int)t->size(1); }
    int ld() const { return (int)t->stride(0); }
    size_t bytes() const { return t ? (size_t)t->numel() * t->element_size() : 0; }
};

int count(const Arg& a) { return a.t ? (a.t->numel() <= INT_MAX ? (int)a.t->numel() : -1) : 0; }
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

// The library call, with the interpreter released for as long as it takes.  Pointers and sizes come as values: reading a
// tensor may throw (a storage that refuses access) and must not run beside other Python threads.
template <class... P>
PyObject* call(int (*entry_point)(P...), std::common_type_t<P>... args) {
    int rc;
    Py_BEGIN_ALLOW_THREADS rc = entry_point(args...);
    Py_END_ALLOW_THREADS return PyLong_FromLong(rc);
}

// linear(kind, x, outlier_idx, weights, w_scale, w_reduced, w_out, bias, out, workspace); kind: 4 or 8 (bits), 84 (4-bit
// weights under 8-bit activations), 6 (FP6), 24 (2:4-sparse)
PyObject* linear(PyObject*, PyObject* const* o, Py_ssize_t n) {
    if (n != 10 || !PyLong_Check(o[0])) Py_RETURN_NONE;
    const long kind = PyLong_AsLong(o[0]);
    if (kind == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const Arg x(o[1]), idx(o[2]), w(o[3]), sw(o[4]), wr(o[5]), wo(o[6]), bias(o[7]), y(o[8]), ws(o[9]);
    const int n_out = idx.ok ? count(idx) : -1;
    if (!(x.ok && idx.ok && w.ok && sw.ok && wr.ok && wo.ok && bias.ok && y.ok && ws.ok) || n_out < 0 || !ws.t ||
        !x.matrix(at::kHalf) || !y.matrix(at::kHalf) || !w.t || w.t->scalar_type() != at::kByte ||
        (n_out && !(idx.vector(at::kInt) && wo.matrix(at::kHalf))) || !sw.vector(at::kHalf) || !wr.vector(at::kFloat) ||
        !bias.vector_or_none(at::kHalf) || !ws.buffer_or_none())
        Py_RETURN_NONE;
    const int T = x.rows(), K = x.cols(), ldwo = n_out ? wo.ld() : 0;
    const void* px = x.ptr();
    const int32_t* pi = n_out ? static_cast<const int32_t*>(idx.ptr()) : nullptr;
    const void* po = n_out ? wo.ptr() : nullptr;
    const float* pr = static_cast<const float*>(wr.ptr());
    void* const st = stream();
    if (kind == 4 || kind == 8 || kind == 84) {
        if (!w.matrix()) Py_RETURN_NONE;
        const int N = w.rows();
        if (kind == 84) {
            return call(entry.linear_w4a8, px, T, K, x.ld(), pi, n_out, w.ptr(), w.ld(), sw.ptr(), pr, po, ldwo, bias.ptr(),
                        N, y.ptr(), y.ld(), ws.ptr(), (size_t)ws.t->numel(), st);
        }
        return call(entry.linear, px, T, K, x.ld(), pi, n_out, (int)kind, w.ptr(), w.ld(), sw.ptr(), pr, po, ldwo,
                    bias.ptr(), N, y.ptr(), y.ld(), ws.ptr(), ws.bytes(), st);
    }
    if (kind != 6 && kind != 24) Py_RETURN_NONE;
    // panels [stages, rows, bytes]
    if (w.t->dim() != 3 || w.t->stride(2) != 1 || w.t->size(1) > INT_MAX || sw.t->numel() > INT_MAX) Py_RETURN_NONE;
    if (kind == 6) {
        return call(entry.linear_fp6, px, T, K, x.ld(), pi, n_out, w.ptr(), sw.ptr(), pr, po, ldwo, bias.ptr(),
                    (int)w.t->size(1), y.ptr(), y.ld(), ws.ptr(), (size_t)ws.t->numel(), st);
    }
    return call(entry.linear_sp24, px, T, K, x.ld(), pi, n_out, w.ptr(), sw.ptr(), pr, po, ldwo, bias.ptr(),
                (int)sw.t->numel(), y.ptr(), y.ld(), ws.ptr(), (size_t)ws.t->numel(), st);
}

// quantize(x, outlier_idx, bits, xq, scale, zero, x_out, workspace)
PyObject* quantize(PyObject*, PyObject* const* o, Py_ssize_t n) {
    if (n != 8 || !PyLong_Check(o[2])) Py_RETURN_NONE;
    const long bits = PyLong_AsLong(o[2]);
    if (bits == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const Arg x(o[0]), idx(o[1]), xq(o[3]), sc(o[4]), ze(o[5]), xo(o[6]), ws(o[7]);
    const int n_out = idx.ok ? count(idx) : -1;
    if (!(x.ok && idx.ok && xq.ok && sc.ok && ze.ok && xo.ok && ws.ok) || n_out < 0 || (bits != 4 && bits != 8) ||
        !x.matrix(at::kHalf) || !xq.matrix(at::kByte) || !sc.vector(at::kFloat) || !ze.vector(at::kFloat) ||
        (n_out && !(idx.vector(at::kInt) && xo.matrix(at::kHalf))) || !ws.buffer_or_none() || n_out >= x.cols() || x.cols() >= 131072 || ((long)(x.cols() - n_out) * bits) % 8)
        Py_RETURN_NONE;
    void* const st = stream();
    return call(entry.quantize, x.ptr(), x.rows(), x.cols(), x.ld(),
                n_out ? static_cast<const int32_t*>(idx.ptr()) : nullptr, n_out, (int)bits, xq.ptr(), xq.ld(),
                static_cast<float*>(sc.ptr()), static_cast<float*>(ze.ptr()), n_out ? xo.ptr() : nullptr,
                n_out ? xo.ld() : 0, ws.ptr(), ws.bytes(), st);
}

// gemm_dequant(xq, scale, zero, x_out, K_b, bits, w_q, w_scale, w_reduced, w_out, bias, out, workspace)
PyObject* gemm_dequant(PyObject*, PyObject* const* o, Py_ssize_t n) {
    if (n != 13 || !PyLong_Check(o[4]) || !PyLong_Check(o[5])) Py_RETURN_NONE;
    const long K_b = PyLong_AsLong(o[4]), bits = PyLong_AsLong(o[5]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const Arg xq(o[0]), sc(o[1]), ze(o[2]), xo(o[3]), w(o[6]), sw(o[7]), wr(o[8]), wo(o[9]), bias(o[10]), y(o[11]), ws(o[12]);
    if (!(xq.ok && sc.ok && ze.ok && xo.ok && w.ok && sw.ok && wr.ok && wo.ok && bias.ok && y.ok && ws.ok) ||
        !xq.matrix(at::kByte) || !w.matrix(at::kByte) || !y.matrix(at::kHalf) || (xo.t && !xo.matrix(at::kHalf)) ||
        !sc.vector(at::kFloat) || !ze.vector(at::kFloat) || !sw.vector(at::kHalf) || !wr.vector(at::kFloat) ||
        !bias.vector_or_none(at::kHalf) || !ws.buffer_or_none() || K_b < INT_MIN || K_b > INT_MAX || bits < INT_MIN ||
        bits > INT_MAX)
        Py_RETURN_NONE;
    const int n_out = xo.t ? xo.cols() : 0;
    if (n_out && !wo.matrix(at::kHalf)) Py_RETURN_NONE;
    void* const st = stream();
    return call(entry.gemm_dequant, xq.ptr(), xq.ld(), static_cast<const float*>(sc.ptr()),
                static_cast<const float*>(ze.ptr()), n_out ? xo.ptr() : nullptr, n_out ? xo.ld() : 0, xq.rows(), (int)K_b,
                n_out, (int)bits, w.ptr(), w.ld(), sw.ptr(), static_cast<const float*>(wr.ptr()), n_out ? wo.ptr() : nullptr,
                n_out ? wo.ld() : 0, bias.ptr(), w.rows(), y.ptr(), y.ld(), ws.ptr(), ws.bytes(), st);
}

// bind(addresses of quik_linear, _w4a8, _fp6, _sp24, quik_quantize, quik_gemm_dequant)
PyObject* bind(PyObject*, PyObject* const* o, Py_ssize_t n) {
    if (n != 6) {
        PyErr_SetString(PyExc_TypeError, "bind takes six addresses");
        return nullptr;
    }
    void** const at[6] = {(void**)&entry.linear,      (void**)&entry.linear_w4a8, (void**)&entry.linear_fp6,
                          (void**)&entry.linear_sp24, (void**)&entry.quantize,    (void**)&entry.gemm_dequant};
    for (int i = 0; i < 6; ++i) {
        *at[i] = PyLong_AsVoidPtr(o[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_RETURN_NONE;
}

// torch's C++ errors become Python's, as in its own bindings
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* o, Py_ssize_t n) {
    try {
        return F(self, o, n);
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

PyMethodDef methods[] = {{"bind", (PyCFunction)(void (*)())bind, METH_FASTCALL, nullptr},
                         {"linear", (PyCFunction)(void (*)())guarded<linear>, METH_FASTCALL, nullptr},
                         {"quantize", (PyCFunction)(void (*)())guarded<quantize>, METH_FASTCALL, nullptr},
                         {"gemm_dequant", (PyCFunction)(void (*)())guarded<gemm_dequant>, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_quik_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// BUILT_FOR: the torch and Python this was compiled for (the binding uses it with these only)
PyMODINIT_FUNC PyInit__quik_call() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "BUILT_FOR", QUIK_BUILT_FOR) < 0) Py_CLEAR(m);
    return m;
}
