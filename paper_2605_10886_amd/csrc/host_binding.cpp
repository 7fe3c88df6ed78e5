// The per-step calls of binding.py as native code: read the tensors, allocate the outputs, take the current stream and
// call the C ABI (include/loka.h).  Nothing is computed here.
//
// Why native: a small layer is two launches of a few microseconds of GPU time, and the same marshalling through ctypes
// (a Python-level allocation per output, a stream object, five to ten boxed pointers per call) took 12 - 14 us of
// host time per call, so the GPU waited for the host.  Positional arguments only; binding.py's wrappers carry the
// keyword interface.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/loka.h"

namespace {

PyObject* g_error = nullptr;       // binding.LokaError

// (status, what) becomes LokaError(status, what)
PyObject* fail(loka_status st, const char* what) {
    PyObject* args = Py_BuildValue("(is)", static_cast<int>(st), what);
    if (args) {
        PyErr_SetObject(g_error ? g_error : PyExc_RuntimeError, args);
        Py_DECREF(args);
    }
    return nullptr;
}

const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) throw std::invalid_argument("expected a tensor");
    return THPVariable_Unpack(o);
}
void* ptr(const at::Tensor& t) { return t.data_ptr(); }
void* ptr_or_null(PyObject* o) { return o == Py_None ? nullptr : tensor(o).data_ptr(); }

at::Tensor empty(at::IntArrayRef size, at::ScalarType type, const at::Device& dev) {
    return at::Tensor(at::detail::empty_cuda(size, type, dev, std::nullopt));
}
// the caller's tensor, or a new one
at::Tensor given_or(PyObject* o, at::IntArrayRef size, at::ScalarType type, const at::Device& dev) {
    return o == Py_None ? empty(size, type, dev) : tensor(o);
}
at::Tensor scratch(size_t bytes, const at::Device& dev) {
    return bytes ? empty({static_cast<int64_t>(bytes)}, at::kByte, dev) : at::Tensor();
}
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

loka_gemm_desc desc_of(PyObject* o) {      // a ctypes structure: its bytes are the descriptor
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        throw std::invalid_argument("expected a GemmDesc");
    }
    loka_gemm_desc d;
    const bool ok = b.len == static_cast<Py_ssize_t>(sizeof(d));
    if (ok) memcpy(&d, b.buf, sizeof(d));
    PyBuffer_Release(&b);
    if (!ok) throw std::invalid_argument("expected a GemmDesc");
    return d;
}

// the library call without the interpreter lock (a launch can block while the hardware queue is full); a tensor without
// storage throws where its pointer is taken, and the lock has to be back before that becomes a Python exception
struct LockReleased {
    PyThreadState* const state = PyEval_SaveThread();
    ~LockReleased() { PyEval_RestoreThread(state); }
};
template <class F>
loka_status unlocked(F&& f) {
    const LockReleased released;
    return f();
}

PyObject* wrap(const at::Tensor& t) {
    if (!t.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(t);
}
PyObject* pack(std::initializer_list<at::Tensor> ts) {
    PyObject* r = PyTuple_New(static_cast<Py_ssize_t>(ts.size()));
    if (!r) return nullptr;
    Py_ssize_t i = 0;
    for (const at::Tensor& t : ts) {
        PyObject* o = wrap(t);
        if (!o) { Py_DECREF(r); return nullptr; }
        PyTuple_SET_ITEM(r, i++, o);
    }
    return r;
}
bool need_args(Py_ssize_t n, Py_ssize_t want) {
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return false;
}

// quantize(x, mode, transpose_out) -> (codes, scales)
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!need_args(n, 3)) return nullptr;
    const at::Tensor& x = tensor(a[0]);
    const long mode_l = PyLong_AsLong(a[1]);
    const int tr = PyObject_IsTrue(a[2]);
    if ((mode_l == -1 && PyErr_Occurred()) || tr < 0) return nullptr;
    if (x.scalar_type() != at::kBFloat16 || x.dim() != 2 || x.stride(1) != 1) {
        PyErr_SetString(PyExc_AssertionError, "x: bf16 [rows, cols] with contiguous rows");
        return nullptr;
    }
    const loka_scale_mode mode = static_cast<loka_scale_mode>(mode_l);
    const int64_t rows = x.size(0), cols = x.size(1), groups = loka_scale_count(mode, rows, cols);
    if (groups < 0) return fail(LOKA_ERR_SHAPE, "loka_scale_count");
    const at::Device dev = x.device();
    at::Tensor q = tr ? empty({cols, rows}, at::kByte, dev) : empty({rows, cols}, at::kByte, dev);
    at::Tensor s = empty({groups}, at::kFloat, dev);
    const size_t bytes = loka_quantize_workspace(mode, rows, cols, tr);
    at::Tensor ws = scratch(bytes, dev);
    void* st_ = stream();
    const loka_status st = unlocked([&] {
        return loka_quantize(ptr(x), rows, cols, x.stride(0), mode, tr, static_cast<uint8_t*>(ptr(q)),
                             static_cast<float*>(ptr(s)), bytes ? ptr(ws) : nullptr, bytes, st_);
    });
    if (st != LOKA_OK) return fail(st, "loka_quantize");
    return pack({q, s});
    END_HANDLE_TH_ERRORS
}

// gemm_norm(desc, xq, sx, wq, sw, gamma, beta, want_y, out, y, workspace) -> (out, y or None)
PyObject* gemm_norm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!need_args(n, 11)) return nullptr;
    const loka_gemm_desc d = desc_of(a[0]);
    const at::Device dev = tensor(a[1]).device();
    const int64_t rows = d.batch * d.M;
    const int want_y = PyObject_IsTrue(a[7]);
    if (want_y < 0) return nullptr;
    at::Tensor out = given_or(a[8], {rows, d.N}, at::kBFloat16, dev);
    at::Tensor y = (want_y || a[9] != Py_None) ? given_or(a[9], {rows, d.N}, at::kFloat, dev) : at::Tensor();
    at::Tensor ws = a[10] == Py_None ? scratch(loka_fp8_gemm_norm_workspace(&d), dev) : tensor(a[10]);
    void* const p[6] = {ptr_or_null(a[1]), ptr_or_null(a[2]), ptr_or_null(a[3]), ptr_or_null(a[4]), ptr_or_null(a[5]), ptr_or_null(a[6])};
    void* st_ = stream();
    const loka_status st = unlocked([&] {
        return loka_fp8_gemm_norm(&d, static_cast<uint8_t*>(p[0]), static_cast<float*>(p[1]), static_cast<uint8_t*>(p[2]),
                                  static_cast<float*>(p[3]), p[4], p[5], ptr(out), y.defined() ? static_cast<float*>(ptr(y)) : nullptr,
                                  ws.defined() ? ptr(ws) : nullptr, ws.defined() ? static_cast<size_t>(ws.numel()) : 0, st_);
    });
    if (st != LOKA_OK) return fail(st, "loka_fp8_gemm_norm");
    return pack({out, y});
    END_HANDLE_TH_ERRORS
}

// gemm_norm_fp8out(desc, xq, sx, wq, sw, gamma, beta, want_y, oq, so, y, workspace) -> (codes, row scales, y or None)
PyObject* gemm_norm_fp8out(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!need_args(n, 12)) return nullptr;
    const loka_gemm_desc d = desc_of(a[0]);
    const at::Device dev = tensor(a[1]).device();
    const int64_t rows = d.batch * d.M;
    const int want_y = PyObject_IsTrue(a[7]);
    if (want_y < 0) return nullptr;
    at::Tensor oq = given_or(a[8], {rows, d.N}, at::kByte, dev);
    at::Tensor so = given_or(a[9], {rows}, at::kFloat, dev);
    at::Tensor y = (want_y || a[10] != Py_None) ? given_or(a[10], {rows, d.N}, at::kFloat, dev) : at::Tensor();
    at::Tensor ws = a[11] == Py_None ? scratch(loka_fp8_gemm_norm_fp8out_workspace(&d), dev) : tensor(a[11]);
    void* const p[6] = {ptr_or_null(a[1]), ptr_or_null(a[2]), ptr_or_null(a[3]), ptr_or_null(a[4]), ptr_or_null(a[5]), ptr_or_null(a[6])};
    void* st_ = stream();
    const loka_status st = unlocked([&] {
        return loka_fp8_gemm_norm_fp8out(&d, static_cast<uint8_t*>(p[0]), static_cast<float*>(p[1]), static_cast<uint8_t*>(p[2]),
                                         static_cast<float*>(p[3]), p[4], p[5], static_cast<uint8_t*>(ptr(oq)),
                                         static_cast<float*>(ptr(so)), y.defined() ? static_cast<float*>(ptr(y)) : nullptr,
                                         ws.defined() ? ptr(ws) : nullptr, ws.defined() ? static_cast<size_t>(ws.numel()) : 0, st_);
    });
    if (st != LOKA_OK) return fail(st, "loka_fp8_gemm_norm_fp8out");
    return pack({oq, so, y});
    END_HANDLE_TH_ERRORS
}

// linear_norm(desc, x, wq, sw, gamma, beta, want_y, want_sx, out) -> (out, y or None, sx or None)
PyObject* linear_norm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!need_args(n, 9)) return nullptr;
    const loka_gemm_desc d = desc_of(a[0]);
    const at::Device dev = tensor(a[1]).device();
    const int64_t rows = d.batch * d.M;
    const int want_y = PyObject_IsTrue(a[6]), want_sx = PyObject_IsTrue(a[7]);
    if (want_y < 0 || want_sx < 0) return nullptr;
    at::Tensor out = given_or(a[8], {rows, d.N}, at::kBFloat16, dev);
    at::Tensor y = want_y ? empty({rows, d.N}, at::kFloat, dev) : at::Tensor();
    at::Tensor sx = want_sx ? empty({rows}, at::kFloat, dev) : at::Tensor();
    void* const p[5] = {ptr_or_null(a[1]), ptr_or_null(a[2]), ptr_or_null(a[3]), ptr_or_null(a[4]), ptr_or_null(a[5])};
    void* st_ = stream();
    const loka_status st = unlocked([&] {
        return loka_fp8_linear_norm(&d, p[0], static_cast<uint8_t*>(p[1]), static_cast<float*>(p[2]), p[3], p[4], ptr(out),
                                    y.defined() ? static_cast<float*>(ptr(y)) : nullptr,
                                    sx.defined() ? static_cast<float*>(ptr(sx)) : nullptr, st_);
    });
    if (st != LOKA_OK) return fail(st, "loka_fp8_linear_norm");
    return pack({out, y, sx});
    END_HANDLE_TH_ERRORS
}

// linear_norm_xq(desc, x, wq, sw, gamma, beta, want_y, out, xq, sx) -> (out, y or None, xq, sx)
PyObject* linear_norm_xq(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!need_args(n, 10)) return nullptr;
    const loka_gemm_desc d = desc_of(a[0]);
    const at::Device dev = tensor(a[1]).device();
    const int64_t rows = d.batch * d.M;
    const int want_y = PyObject_IsTrue(a[6]);
    if (want_y < 0) return nullptr;
    at::Tensor out = given_or(a[7], {rows, d.N}, at::kBFloat16, dev);
    at::Tensor xq = given_or(a[8], {rows, d.K}, at::kByte, dev);
    at::Tensor sx = given_or(a[9], {rows}, at::kFloat, dev);
    at::Tensor y = want_y ? empty({rows, d.N}, at::kFloat, dev) : at::Tensor();
    void* const p[5] = {ptr_or_null(a[1]), ptr_or_null(a[2]), ptr_or_null(a[3]), ptr_or_null(a[4]), ptr_or_null(a[5])};
    void* st_ = stream();
    const loka_status st = unlocked([&] {
        return loka_fp8_linear_norm_xq(&d, p[0], static_cast<uint8_t*>(ptr(xq)), static_cast<float*>(ptr(sx)),
                                       static_cast<uint8_t*>(p[1]), static_cast<float*>(p[2]), p[3], p[4], ptr(out),
                                       y.defined() ? static_cast<float*>(ptr(y)) : nullptr, st_);
    });
    if (st != LOKA_OK) return fail(st, "loka_fp8_linear_norm_xq");
    return pack({out, y, xq, sx});
    END_HANDLE_TH_ERRORS
}

// bf16_gemm(desc, x, w, yref, workspace) -> yref
PyObject* bf16_gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!need_args(n, 5)) return nullptr;
    loka_gemm_desc d = desc_of(a[0]);
    if (d.strideW) d.strideW = d.K * d.N;           // the weights lie as [batch][K, N] here
    const at::Device dev = tensor(a[1]).device();
    at::Tensor yref = given_or(a[3], {d.batch * d.M, d.N}, at::kFloat, dev);
    at::Tensor ws = a[4] == Py_None ? scratch(loka_bf16_gemm_workspace(&d), dev) : tensor(a[4]);
    void* const p[2] = {ptr_or_null(a[1]), ptr_or_null(a[2])};
    void* st_ = stream();
    const loka_status st = unlocked([&] {
        return loka_bf16_gemm(&d, p[0], p[1], static_cast<float*>(ptr(yref)), ws.defined() ? ptr(ws) : nullptr,
                              ws.defined() ? static_cast<size_t>(ws.numel()) : 0, st_);
    });
    if (st != LOKA_OK) return fail(st, "loka_bf16_gemm");
    return wrap(yref);
    END_HANDLE_TH_ERRORS
}

// probe_error(y, yref, stats, rowmax, workspace) -> (stats, rowmax)
PyObject* probe_error(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!need_args(n, 5)) return nullptr;
    const at::Tensor& y = tensor(a[0]);
    const at::Tensor& yref = tensor(a[1]);
    if (y.scalar_type() != at::kFloat || yref.scalar_type() != at::kFloat || y.dim() != 2 || !y.sizes().equals(yref.sizes())) {
        PyErr_SetString(PyExc_AssertionError, "y, yref: fp32 [M, N] of one shape");
        return nullptr;
    }
    const at::Device dev = y.device();
    const int64_t M = y.size(0), N = y.size(1);
    at::Tensor stats = given_or(a[2], {5}, at::kDouble, dev);
    at::Tensor rowmax = given_or(a[3], {M}, at::kFloat, dev);
    at::Tensor ws = a[4] == Py_None ? scratch(loka_probe_error_workspace(M, N), dev) : tensor(a[4]);
    void* st_ = stream();
    const loka_status st = unlocked([&] {
        return loka_probe_error(static_cast<float*>(ptr(y)), static_cast<float*>(ptr(yref)), M, N, y.stride(0),
                                static_cast<loka_probe_stats*>(ptr(stats)), static_cast<float*>(ptr(rowmax)),
                                ws.defined() ? ptr(ws) : nullptr, ws.defined() ? static_cast<size_t>(ws.numel()) : 0, st_);
    });
    if (st != LOKA_OK) return fail(st, "loka_probe_error");
    return pack({stats, rowmax});
    END_HANDLE_TH_ERRORS
}

// tracker_update(x, n_old, mu, sigma, workspace) -> n_old + rows of x
PyObject* tracker_update(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!need_args(n, 5)) return nullptr;
    const at::Tensor& x = tensor(a[0]);
    if (x.dim() != 2) {
        PyErr_SetString(PyExc_ValueError, "x: [rows, features]");
        return nullptr;
    }
    const long long n_old = PyLong_AsLongLong(a[1]);
    if (n_old == -1 && PyErr_Occurred()) return nullptr;
    const int64_t rows = x.size(0), K = x.size(1);
    at::Tensor ws = a[4] == Py_None ? scratch(loka_tracker_update_workspace(rows, K), x.device()) : tensor(a[4]);
    void* const p[2] = {ptr_or_null(a[2]), ptr_or_null(a[3])};
    void* st_ = stream();
    const loka_status st = unlocked([&] {
        return loka_tracker_update(ptr(x), rows, K, x.stride(0), n_old, static_cast<float*>(p[0]), static_cast<float*>(p[1]),
                                   ws.defined() ? ptr(ws) : nullptr, ws.defined() ? static_cast<size_t>(ws.numel()) : 0, st_);
    });
    if (st != LOKA_OK) return fail(st, "loka_tracker_update");
    return PyLong_FromLongLong(n_old + rows);
    END_HANDLE_TH_ERRORS
}

PyObject* set_error(PyObject*, PyObject* cls) {
    Py_INCREF(cls);
    Py_XSETREF(g_error, cls);
    Py_RETURN_NONE;
}

#define LOKA_FAST(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&NAME)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    LOKA_FAST(quantize), LOKA_FAST(gemm_norm), LOKA_FAST(gemm_norm_fp8out), LOKA_FAST(linear_norm), LOKA_FAST(linear_norm_xq),
    LOKA_FAST(bf16_gemm), LOKA_FAST(probe_error), LOKA_FAST(tracker_update),
    {"set_error", &set_error, METH_O, "the exception class raised for a status other than LOKA_OK"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_host", "marshalling of the per-step calls", -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host(void) { return PyModule_Create(&kModule); }
