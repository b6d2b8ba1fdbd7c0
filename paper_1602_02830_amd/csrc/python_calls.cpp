// Direct calls from Python into the C ABI, for the case every loop of a program is in: tensors that fit, and an output
// that exists.  Each function takes the arguments of the wrapper of the same name in binding.py, checks what that
// wrapper checks, reads pointers and strides off the tensors and calls the library on torch's current stream.
//
//   returns 0    launched
//   returns > 0  the library's status (nothing launched)
//   returns -1   not a case for this path (another type, a tensor subclass or wrapper, a shape or stride that the
//                wrapper refuses): nothing was done, and the wrapper's own checks say what is wrong or go the long way
//
// Why it exists: with attribute reads, checks and a foreign call through ctypes a launch from Python took 6 - 8 us, twice
// what the GPU needs for a small layer (64 x 1024 x 1024 fused: 3.0 us).  Here it takes about 0.6 us.
//
// The library is loaded by binding.py, which hands over the entry points' addresses (bind); nothing is kept of a tensor
// after a call.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

using Words = const uint32_t*;

struct EntryPoints {
    int (*pack_sign)(const float*, int64_t, int64_t, int64_t, uint32_t*, int64_t, void*);
    int (*xnor_gemm)(Words, int64_t, Words, int64_t, int32_t*, int64_t, int64_t, int64_t, int64_t, void*);
    int (*xnor_gemm_kernel)(Words, int64_t, Words, int64_t, int32_t*, int64_t, int64_t, int64_t, int64_t, int, void*);
    int (*bn_sign_pack)(const int32_t*, int64_t, int64_t, int64_t, const int32_t*, Words, uint32_t*, int64_t, void*);
    int (*xnor_gemm_bn_sign_pack)(Words, int64_t, Words, int64_t, int64_t, int64_t, int64_t, const int32_t*, Words, uint32_t*,
                                  int64_t, void*);
    int (*xnor_gemm_bn_sign_pack_kernel)(Words, int64_t, Words, int64_t, int64_t, int64_t, int64_t, const int32_t*, Words,
                                         uint32_t*, int64_t, int, void*);
    int (*sign_gemm_bn_sign_pack)(const float*, int64_t, Words, int64_t, int64_t, int64_t, int64_t, const int32_t*, Words, uint32_t*,
                                  int64_t, uint32_t*, int64_t, void*);
    int (*pack_bitplanes)(const uint8_t*, int64_t, int64_t, int64_t, uint32_t*, int64_t, void*);
    int (*bitplane_gemm)(Words, int64_t, Words, int64_t, int32_t*, int64_t, int64_t, int64_t, int64_t, void*);
    int (*bitplane_gemm_bn_sign_pack)(Words, int64_t, Words, int64_t, int64_t, int64_t, int64_t, const int32_t*, Words,
                                      uint32_t*, int64_t, void*);
    int (*conv_xnor)(Words, int64_t, int64_t, int64_t, int64_t, Words, int64_t, int64_t, int, int, int, int, int32_t*, int64_t,
                     void*);
    int (*conv_bn_sign_pack)(Words, int64_t, int64_t, int64_t, int64_t, Words, int64_t, int64_t, int, int, int, int,
                             const int32_t*, Words, uint32_t*, int64_t, void*);
    int (*conv_pool_bn_sign_pack)(Words, int64_t, int64_t, int64_t, int64_t, Words, int64_t, int64_t, int, int, int, int, int,
                                  const int32_t*, Words, uint32_t*, int64_t, void*);
    int (*conv_pool_windows_bn_sign_pack)(Words, int64_t, int64_t, int64_t, int64_t, Words, int64_t, int64_t, int, int, int, int, int,
                                          const int32_t*, Words, uint32_t*, int64_t, void*);
    int (*conv_im2col_pack)(Words, int64_t, int64_t, int64_t, int64_t, int, int, int, int, uint32_t*, int64_t, void*);
    int (*maxpool_bits)(Words, int64_t, int64_t, int64_t, int64_t, int, int, int, Words, uint32_t*, void*);
};

EntryPoints entry{};
PyObject* raw_stream = nullptr;      // torch._C._cuda_getCurrentRawStream

int64_t words(int64_t n) { return (n + 31) / 32; }

// A plain torch.Tensor on the GPU with memory of its own, of the given type; null otherwise.
const at::Tensor* plain(PyObject* o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || t.layout() != at::kStrided ||
        !t.unsafeGetTensorImpl()->has_storage())
        return nullptr;
    return &t;
}

// The wrappers' 2-D operand: unit stride along its rows.
struct Matrix {
    void* data = nullptr;
    int64_t rows = 0, cols = 0, ld = 0;
    const at::Tensor* t = nullptr;
    bool read(PyObject* o, at::ScalarType type) {
        t = plain(o, type);
        if (!t || t->dim() != 2) return false;
        rows = t->size(0);
        cols = t->size(1);
        if (cols > 1 && t->stride(1) != 1) return false;
        ld = rows > 1 ? t->stride(0) : std::max(t->stride(0), cols);
        data = t->data_ptr();
        return true;
    }
    template <typename T>
    T* as() const { return static_cast<T*>(data); }
    // The [r][c] elements a call reads or writes are there.  A leading dimension that is too short is left to the library,
    // which refuses it; too few rows, or a narrow slice of a wide buffer, it cannot see.
    bool holds(int64_t r, int64_t c) const { return r <= 0 || c <= 0 || ld < c || (rows >= r && cols >= c); }
};

// A packed map [B][H][W][words], contiguous.
struct Map {
    Words data = nullptr;
    int64_t B = 0, H = 0, W = 0, Cw = 0;
    bool read(PyObject* o, int64_t channels) {
        const at::Tensor* t = plain(o, at::kInt);
        if (!t || t->dim() != 4 || !t->is_contiguous()) return false;
        B = t->size(0);
        H = t->size(1);
        W = t->size(2);
        Cw = t->size(3);
        data = static_cast<Words>(t->data_ptr());
        return Cw == words(channels);
    }
};

// Contiguous int32 vector of n elements.
void* vector_of(PyObject* o, int64_t n) {
    const at::Tensor* t = plain(o, at::kInt);
    return t && t->numel() == n && t->is_contiguous() ? t->data_ptr() : nullptr;
}

bool integer(PyObject* o, int64_t& v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}

bool small_integer(PyObject* o, int& v) {
    int64_t w;
    if (!integer(o, w) || w < -1000000000 || w > 1000000000) return false;
    v = int(w);
    return true;
}

bool stream_of(const at::Tensor& t, void*& stream) {
    PyObject* index = PyLong_FromLong(t.get_device());
    if (!index) return false;
    PyObject* r = PyObject_CallOneArg(raw_stream, index);
    Py_DECREF(index);
    if (!r) return false;
    stream = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

PyObject* long_way() { return PyLong_FromLong(-1); }

// Calls the library without the interpreter lock (a launch may wait for room in the stream's queue).
template <typename F>
PyObject* launch(const at::Tensor& out, F&& call) {
    void* stream;
    if (!stream_of(out, stream)) return nullptr;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call(stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// Every function below: no C++ exception may reach the interpreter; whatever a tensor throws is left to the wrapper.
template <PyObject* (*F)(PyObject* const*)>
PyObject* guarded(PyObject* const* a) noexcept {
    try {
        return F(a);
    } catch (...) {
        PyErr_Clear();
        return long_way();
    }
}

template <PyObject* (*F)(PyObject* const*), Py_ssize_t ARGS>
PyObject* entry_of(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != ARGS) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    return guarded<F>(a);
}

// (x, out)
PyObject* pack_sign(PyObject* const* a) {
    Matrix x, out;
    if (!x.read(a[0], at::kFloat) || !out.read(a[1], at::kInt) || !out.holds(x.rows, words(x.cols))) return long_way();
    return launch(*out.t, [&](void* s) { return entry.pack_sign(x.as<float>(), x.rows, x.cols, x.ld, out.as<uint32_t>(), out.ld, s); });
}

// (A, B, K, out, kernel)
PyObject* xnor_gemm(PyObject* const* a) {
    Matrix A, B, out;
    int64_t K;
    int kernel;
    if (!A.read(a[0], at::kInt) || !B.read(a[1], at::kInt) || !integer(a[2], K) || !out.read(a[3], at::kInt) ||
        !small_integer(a[4], kernel) || K < 0 || A.cols < words(K) || B.cols < words(K) || !out.holds(A.rows, B.rows))
        return long_way();
    return launch(*out.t, [&](void* s) {
        return kernel == 0 ? entry.xnor_gemm(A.as<uint32_t>(), A.ld, B.as<uint32_t>(), B.ld, out.as<int32_t>(), out.ld, A.rows,
                                             B.rows, K, s)
                           : entry.xnor_gemm_kernel(A.as<uint32_t>(), A.ld, B.as<uint32_t>(), B.ld, out.as<int32_t>(), out.ld,
                                                    A.rows, B.rows, K, kernel, s);
    });
}

// (C, thr, flip, out)
PyObject* bn_sign_pack(PyObject* const* a) {
    Matrix C, out;
    if (!C.read(a[0], at::kInt)) return long_way();
    const void* thr = vector_of(a[1], C.cols);
    const void* flip = vector_of(a[2], words(C.cols));
    if (!thr || !flip || !out.read(a[3], at::kInt) || !out.holds(C.rows, words(C.cols))) return long_way();
    return launch(*out.t, [&](void* s) {
        return entry.bn_sign_pack(C.as<int32_t>(), C.ld, C.rows, C.cols, static_cast<const int32_t*>(thr),
                                  static_cast<Words>(flip), out.as<uint32_t>(), out.ld, s);
    });
}

// (A, B, K, thr, flip, out, kernel)
PyObject* xnor_gemm_bn_sign_pack(PyObject* const* a) {
    Matrix A, B, out;
    int64_t K;
    int kernel;
    if (!A.read(a[0], at::kInt) || !B.read(a[1], at::kInt) || !integer(a[2], K) || K < 0 || A.cols < words(K) ||
        B.cols < words(K))
        return long_way();
    const void* thr = vector_of(a[3], B.rows);
    const void* flip = vector_of(a[4], words(B.rows));
    if (!thr || !flip || !out.read(a[5], at::kInt) || !small_integer(a[6], kernel) || !out.holds(A.rows, words(B.rows)))
        return long_way();
    return launch(*out.t, [&](void* s) {
        return kernel == 0
                   ? entry.xnor_gemm_bn_sign_pack(A.as<uint32_t>(), A.ld, B.as<uint32_t>(), B.ld, A.rows, B.rows, K,
                                                  static_cast<const int32_t*>(thr), static_cast<Words>(flip),
                                                  out.as<uint32_t>(), out.ld, s)
                   : entry.xnor_gemm_bn_sign_pack_kernel(A.as<uint32_t>(), A.ld, B.as<uint32_t>(), B.ld, A.rows, B.rows, K,
                                                         static_cast<const int32_t*>(thr), static_cast<Words>(flip),
                                                         out.as<uint32_t>(), out.ld, kernel, s);
    });
}

// (x, B, K, thr, flip, a_bits, out): every row of x is a row of a_bits, and K elements long
PyObject* sign_gemm_bn_sign_pack(PyObject* const* a) {
    Matrix x, B, bits, out;
    int64_t K;
    if (!x.read(a[0], at::kFloat) || !B.read(a[1], at::kInt) || !integer(a[2], K) || K <= 0 || x.cols != K || B.cols < words(K))
        return long_way();
    const void* thr = vector_of(a[3], B.rows);
    const void* flip = vector_of(a[4], words(B.rows));
    if (!thr || !flip || !bits.read(a[5], at::kInt) || bits.rows != x.rows || bits.cols < words(K) || !out.read(a[6], at::kInt) ||
        !out.holds(x.rows, words(B.rows)))
        return long_way();
    return launch(*out.t, [&](void* s) {
        return entry.sign_gemm_bn_sign_pack(x.as<float>(), x.ld, B.as<uint32_t>(), B.ld, x.rows, B.rows, K,
                                            static_cast<const int32_t*>(thr), static_cast<Words>(flip), bits.as<uint32_t>(), bits.ld,
                                            out.as<uint32_t>(), out.ld, s);
    });
}

// (x, out)
PyObject* pack_bitplanes(PyObject* const* a) {
    Matrix x, out;
    if (!x.read(a[0], at::kByte) || !out.read(a[1], at::kInt) || !out.holds(x.rows, 8 * words(x.cols))) return long_way();
    return launch(*out.t, [&](void* s) { return entry.pack_bitplanes(x.as<uint8_t>(), x.rows, x.cols, x.ld, out.as<uint32_t>(), out.ld, s); });
}

// The operands of a product on bit planes, where there is one.
bool planes_hold(const Matrix& X, const Matrix& B, int64_t K) {
    return X.holds(B.rows > 0 ? X.rows : 0, 8 * words(K)) && B.holds(X.rows > 0 ? B.rows : 0, words(K));
}

// (Xp, B, K, out)
PyObject* bitplane_gemm(PyObject* const* a) {
    Matrix X, B, out;
    int64_t K;
    if (!X.read(a[0], at::kInt) || !B.read(a[1], at::kInt) || !integer(a[2], K) || !out.read(a[3], at::kInt) ||
        !planes_hold(X, B, K) || !out.holds(X.rows, B.rows))
        return long_way();
    return launch(*out.t, [&](void* s) {
        return entry.bitplane_gemm(X.as<uint32_t>(), X.ld, B.as<uint32_t>(), B.ld, out.as<int32_t>(), out.ld, X.rows, B.rows, K, s);
    });
}

// (Xp, B, K, thr, flip, out)
PyObject* bitplane_gemm_bn_sign_pack(PyObject* const* a) {
    Matrix X, B, out;
    int64_t K;
    if (!X.read(a[0], at::kInt) || !B.read(a[1], at::kInt) || !integer(a[2], K) || !planes_hold(X, B, K)) return long_way();
    const void* thr = vector_of(a[3], B.rows);
    const void* flip = vector_of(a[4], words(B.rows));
    if (!thr || !flip || !out.read(a[5], at::kInt) || !out.holds(X.rows, words(B.rows))) return long_way();
    return launch(*out.t, [&](void* s) {
        return entry.bitplane_gemm_bn_sign_pack(X.as<uint32_t>(), X.ld, B.as<uint32_t>(), B.ld, X.rows, B.rows, K,
                                                static_cast<const int32_t*>(thr), static_cast<Words>(flip), out.as<uint32_t>(),
                                                out.ld, s);
    });
}

// Output pixels of a convolution; 0 for a geometry that the library refuses.
int64_t conv_pixels(const Map& x, int kh, int kw, int stride, int pad) {
    const int64_t dh = x.H + 2 * int64_t(pad) - kh, dw = x.W + 2 * int64_t(pad) - kw;
    return dh < 0 || dw < 0 ? 0 : x.B * (dh / stride + 1) * (dw / stride + 1);
}

struct Conv {
    Map x;
    Matrix w;
    int64_t Cin = 0, M = 0;
    int kh = 0, kw = 0, stride = 0, pad = 0;
    // (x_bits, Cin, w_bits, kh, kw, stride, pad)
    bool read(PyObject* const* a) {
        if (!integer(a[1], Cin) || Cin <= 0 || !x.read(a[0], Cin) || !w.read(a[2], at::kInt) || !small_integer(a[3], kh) ||
            !small_integer(a[4], kw) || !small_integer(a[5], stride) || !small_integer(a[6], pad) || stride < 1)
            return false;
        M = conv_pixels(x, kh, kw, stride, pad);
        // (a window whose bits do not fit 64 is the wrapper's and the library's to refuse)
        return kh > 0 && kw > 0 && Cin <= INT32_MAX && int64_t(kh) * kw <= INT32_MAX &&
               w.holds(M > 0 ? w.rows : 0, words(int64_t(kh) * kw * Cin));
    }
};

// (x_bits, Cin, w_bits, kh, kw, stride, pad, out)
PyObject* conv_xnor(PyObject* const* a) {
    Conv c;
    Matrix out;
    if (!c.read(a) || !out.read(a[7], at::kInt) || !out.holds(c.M, c.w.rows)) return long_way();
    return launch(*out.t, [&](void* s) {
        return entry.conv_xnor(c.x.data, c.x.B, c.x.H, c.x.W, c.Cin, c.w.as<uint32_t>(), c.w.ld, c.w.rows, c.kh, c.kw, c.stride,
                               c.pad, out.as<int32_t>(), out.ld, s);
    });
}

// (x_bits, Cin, w_bits, kh, kw, stride, pad, thr, flip, out)
PyObject* conv_bn_sign_pack(PyObject* const* a) {
    Conv c;
    Matrix out;
    if (!c.read(a)) return long_way();
    const void* thr = vector_of(a[7], c.w.rows);
    const void* flip = vector_of(a[8], words(c.w.rows));
    if (!thr || !flip || !out.read(a[9], at::kInt) || !out.holds(c.M, words(c.w.rows))) return long_way();
    return launch(*out.t, [&](void* s) {
        return entry.conv_bn_sign_pack(c.x.data, c.x.B, c.x.H, c.x.W, c.Cin, c.w.as<uint32_t>(), c.w.ld, c.w.rows, c.kh, c.kw,
                                       c.stride, c.pad, static_cast<const int32_t*>(thr), static_cast<Words>(flip),
                                       out.as<uint32_t>(), out.ld, s);
    });
}

// (x_bits, Cin, w_bits, kh, kw, stride, pad, thr, flip, out, pool)
template <auto EntryPoints::*POOLED>
PyObject* conv_pool_of(PyObject* const* a) {
    Conv c;
    Matrix out;
    int pool;
    if (!c.read(a) || !small_integer(a[10], pool) || pool < 1) return long_way();
    const void* thr = vector_of(a[7], c.w.rows);
    const void* flip = vector_of(a[8], words(c.w.rows));
    const int64_t dh = c.x.H + 2 * int64_t(c.pad) - c.kh, dw = c.x.W + 2 * int64_t(c.pad) - c.kw;
    if (!thr || !flip || !out.read(a[9], at::kInt) || dh < 0 || dw < 0) return long_way();
    const int64_t Ho = dh / c.stride + 1, Wo = dw / c.stride + 1;
    if (out.rows != c.x.B * (Ho / pool) * (Wo / pool) || out.cols != words(c.w.rows)) return long_way();
    return launch(*out.t, [&](void* s) {
        return (entry.*POOLED)(c.x.data, c.x.B, c.x.H, c.x.W, c.Cin, c.w.as<uint32_t>(), c.w.ld, c.w.rows, c.kh, c.kw,
                               c.stride, c.pad, pool, static_cast<const int32_t*>(thr), static_cast<Words>(flip),
                               out.as<uint32_t>(), out.ld, s);
    });
}
PyObject* conv_pool_bn_sign_pack(PyObject* const* a) { return conv_pool_of<&EntryPoints::conv_pool_bn_sign_pack>(a); }
PyObject* conv_pool_windows_bn_sign_pack(PyObject* const* a) {
    return conv_pool_of<&EntryPoints::conv_pool_windows_bn_sign_pack>(a);
}

// (x_bits, Cin, kh, kw, stride, pad, out)
PyObject* conv_im2col_pack(PyObject* const* a) {
    Map x;
    Matrix out;
    int64_t Cin;
    int kh, kw, stride, pad;
    if (!integer(a[1], Cin) || Cin <= 0 || !x.read(a[0], Cin) || !small_integer(a[2], kh) || !small_integer(a[3], kw) ||
        !small_integer(a[4], stride) || !small_integer(a[5], pad) || stride < 1 || !out.read(a[6], at::kInt) || kh < 1 || kw < 1 ||
        Cin > INT32_MAX || int64_t(kh) * kw > INT32_MAX ||
        !out.holds(conv_pixels(x, kh, kw, stride, pad), words(int64_t(kh) * kw * Cin)))
        return long_way();
    return launch(*out.t, [&](void* s) {
        return entry.conv_im2col_pack(x.data, x.B, x.H, x.W, Cin, kh, kw, stride, pad, out.as<uint32_t>(), out.ld, s);
    });
}

// (x_bits, C, flip or None, ph, pw, stride, out)
PyObject* maxpool_bits(PyObject* const* a) {
    Map x;
    int64_t C;
    int ph, pw, stride;
    if (!integer(a[1], C) || C <= 0 || !x.read(a[0], C) || !small_integer(a[3], ph) || !small_integer(a[4], pw) ||
        !small_integer(a[5], stride) || stride < 1 || x.H < ph || x.W < pw)
        return long_way();
    const void* flip = a[2] == Py_None ? nullptr : vector_of(a[2], x.Cw);
    const at::Tensor* out = plain(a[6], at::kInt);
    if ((a[2] != Py_None && !flip) || !out || !out->is_contiguous() ||
        out->numel() != x.B * ((x.H - ph) / stride + 1) * ((x.W - pw) / stride + 1) * x.Cw)
        return long_way();
    return launch(*out, [&](void* s) {
        return entry.maxpool_bits(x.data, x.B, x.H, x.W, C, ph, pw, stride, static_cast<Words>(flip),
                                  static_cast<uint32_t*>(out->data_ptr()), s);
    });
}

// bind({"bnn_pack_sign": address, ...}, raw_stream)
PyObject* bind(PyObject*, PyObject* args) {
    PyObject *table, *stream;
    if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &table, &stream)) return nullptr;
    EntryPoints e{};
    bool ok = true;
    auto set = [&](auto& fn, const char* name) {
        PyObject* v = PyDict_GetItemString(table, name);
        void* p = v ? PyLong_AsVoidPtr(v) : nullptr;
        if (!p) ok = false;
        fn = reinterpret_cast<std::decay_t<decltype(fn)>>(p);
    };
    set(e.pack_sign, "bnn_pack_sign");
    set(e.xnor_gemm, "bnn_xnor_gemm");
    set(e.xnor_gemm_kernel, "bnn_xnor_gemm_kernel");
    set(e.bn_sign_pack, "bnn_bn_sign_pack");
    set(e.xnor_gemm_bn_sign_pack, "bnn_xnor_gemm_bn_sign_pack");
    set(e.xnor_gemm_bn_sign_pack_kernel, "bnn_xnor_gemm_bn_sign_pack_kernel");
    set(e.sign_gemm_bn_sign_pack, "bnn_sign_gemm_bn_sign_pack");
    set(e.pack_bitplanes, "bnn_pack_bitplanes");
    set(e.bitplane_gemm, "bnn_bitplane_gemm");
    set(e.bitplane_gemm_bn_sign_pack, "bnn_bitplane_gemm_bn_sign_pack");
    set(e.conv_xnor, "bnn_conv_xnor");
    set(e.conv_bn_sign_pack, "bnn_conv_bn_sign_pack");
    set(e.conv_pool_bn_sign_pack, "bnn_conv_pool_bn_sign_pack");
    set(e.conv_pool_windows_bn_sign_pack, "bnn_conv_pool_windows_bn_sign_pack");
    set(e.conv_im2col_pack, "bnn_conv_im2col_pack");
    set(e.maxpool_bits, "bnn_maxpool_bits");
    if (!ok || !PyCallable_Check(stream)) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "an entry point or the stream function is missing");
        return nullptr;
    }
    entry = e;
    Py_INCREF(stream);
    Py_XDECREF(raw_stream);
    raw_stream = stream;
    Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject* const*), Py_ssize_t ARGS>
PyMethodDef fast(const char* name) {
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry_of<F, ARGS>)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    fast<pack_sign, 2>("pack_sign"),
    fast<xnor_gemm, 5>("xnor_gemm"),
    fast<bn_sign_pack, 4>("bn_sign_pack"),
    fast<xnor_gemm_bn_sign_pack, 7>("xnor_gemm_bn_sign_pack"),
    fast<sign_gemm_bn_sign_pack, 7>("sign_gemm_bn_sign_pack"),
    fast<pack_bitplanes, 2>("pack_bitplanes"),
    fast<bitplane_gemm, 4>("bitplane_gemm"),
    fast<bitplane_gemm_bn_sign_pack, 6>("bitplane_gemm_bn_sign_pack"),
    fast<conv_xnor, 8>("conv_xnor"),
    fast<conv_bn_sign_pack, 10>("conv_bn_sign_pack"),
    fast<conv_pool_bn_sign_pack, 11>("conv_pool_bn_sign_pack"),
    fast<conv_pool_windows_bn_sign_pack, 11>("conv_pool_windows_bn_sign_pack"),
    fast<conv_im2col_pack, 7>("conv_im2col_pack"),
    fast<maxpool_bits, 7>("maxpool_bits"),
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", "Direct calls of the bnn C ABI on torch tensors.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
