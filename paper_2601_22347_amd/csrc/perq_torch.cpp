// The device entry points of binding.py as a Python extension module: argument checks, output allocation and the
// call into libperq.so without an interpreter step or a ctypes conversion in between.
//
// A call on a small batch is over on the device in 3 - 6 us, so the host's time is the call's time: 16 rows of
// d = 4096 with a prepared permutation took 9.2 us through ctypes and torch.empty (launch 3.6, two allocations 2.8,
// the rest conversions) and take 5.0 through here.  The module holds no state and no reference; the interpreter's
// lock is released around the library call, as ctypes does.  Names and messages of errors are binding.py's.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/StreamGuard.h>
#include <c10/hip/HIPStream.h>

#include "perq.h"

namespace {

// The Python object's own error, already set.
struct PythonError {};

int64_t integer(PyObject* o) {
    PyObject* const l = PyLong_Check(o) ? Py_NewRef(o) : PyNumber_Long(o);      // as int(o)
    if (l == nullptr) throw PythonError();
    const long long v = PyLong_AsLongLong(l);
    Py_DECREF(l);
    if (v == -1 && PyErr_Occurred()) throw PythonError();
    return v;
}

const at::Tensor& tensor(PyObject* o, const char* what) {
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a tensor, not %s", what, Py_TYPE(o)->tp_name);
        throw PythonError();
    }
    return THPVariable_Unpack(o);
}

// Device address of a tensor, of anything else with a data_ptr(), or null for None.
void* address(PyObject* o) {
    if (o == Py_None) return nullptr;
    if (THPVariable_Check(o)) return THPVariable_Unpack(o).data_ptr();
    PyObject* const v = PyObject_CallMethod(o, "data_ptr", nullptr);
    if (v == nullptr) throw PythonError();
    const auto p = static_cast<uintptr_t>(integer(v));
    Py_DECREF(v);
    return reinterpret_cast<void*>(p);
}

// The stream handed over, or the current one of the current device.
struct Stream {
    void* raw;
    bool given;
};

Stream stream_of(PyObject* o) {
    if (o == Py_None) return {c10::hip::getCurrentHIPStream().stream(), false};
    PyObject* const v = PyObject_GetAttrString(o, "cuda_stream");
    if (v == nullptr) throw PythonError();
    const auto p = static_cast<uintptr_t>(integer(v));
    Py_DECREF(v);
    return {reinterpret_cast<void*>(p), true};
}

struct Rows {
    const uint16_t* x;
    int64_t T, d, ldx;
    at::Device device;
};

Rows rows_of(PyObject* o) {
    const at::Tensor& x = tensor(o, "x");
    if (!x.is_cuda() || x.dim() != 2 || x.stride(1) != 1 || x.element_size() != 2) {
        PyErr_SetString(PyExc_ValueError, "x must be a 2-D CUDA tensor of 16-bit elements with unit column stride");
        throw PythonError();
    }
    const auto type = x.scalar_type();
    if (type != at::kBFloat16 && type != at::kShort && type != at::kUInt16) {
        PyErr_SetString(PyExc_ValueError, "x must hold bf16 values (dtype bfloat16, or int16/uint16 bit patterns)");
        throw PythonError();
    }
    return {static_cast<const uint16_t*>(x.data_ptr()), x.size(0), x.size(1), x.stride(0), x.device()};
}

// The buffers of a call belong to the stream that it runs on.  The allocator hands a block out again as soon as the
// work queued so far on the block's own stream allows it, so one that the current stream owned could be written by the
// call while earlier work of the current stream still used it, and (workspaces, which end with the call) be handed
// out again while the call still ran.  Results are for the current stream too: freed later, they are not used again
// before what it has queued by then is done.
//   Through the dispatcher (at::empty) a buffer takes 0.8 us of the host, from the function that it comes to 0.55: 0.4 us
// of a small call's 5.4 (two buffers; calls of 16 rows 5.42 -> 5.03).  Where a mode of the dispatcher is on (fake tensors,
// functorch, functionalization, tracing), the mode has to see the allocation, as it always did.
at::Tensor buffer(at::IntArrayRef shape, at::ScalarType type, at::Device device, const Stream& stream, bool is_result) {
    const auto empty = [&]() -> at::Tensor {
        const c10::DispatchKeySet modes({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::PythonDispatcher,
                                         c10::DispatchKey::Functionalize, c10::DispatchKey::FuncTorchDynamicLayerFrontMode, c10::DispatchKey::Tracer});
        if (!device.is_cuda() || c10::impl::tls_local_dispatch_key_set().included_.has_any(modes))
            return at::empty(shape, at::TensorOptions().dtype(type).device(device));
        return at::detail::empty_cuda(shape, type, device, std::nullopt);
    };
    if (!stream.given || !device.is_cuda()) return empty();
    const auto current = c10::hip::getCurrentHIPStream(device.index());
    if (current.stream() == stream.raw) return empty();
    const auto on_device = [&](c10::StreamId id) { return c10::Stream(c10::Stream::UNSAFE, device, id); };
    const c10::StreamGuard guard(on_device(c10::hip::getStreamFromExternal(static_cast<hipStream_t>(stream.raw), device.index()).id()));
    at::Tensor t = empty();
    if (is_result) t.record_stream(on_device(current.id()));
    return t;
}

// The library call without the interpreter's lock.
template <typename F>
perq_status_t unlocked(F&& f) {
    perq_status_t st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    return st;
}

// What the Python side gets: the result, or the status of a call that failed.
PyObject* result(perq_status_t st, PyObject* out) {
    if (st == PERQ_OK) return out;
    Py_XDECREF(out);
    return PyLong_FromLong(st);
}

// `given`, or a new buffer.
PyObject* output(PyObject* given, at::IntArrayRef shape, at::ScalarType type, at::Device device, const Stream& stream) {
    return given != Py_None ? Py_NewRef(given) : THPVariable_Wrap(buffer(shape, type, device, stream, true));
}

struct Held {
    PyObject* o;
    explicit Held(PyObject* p) : o(p) {
        if (p == nullptr) throw PythonError();
    }
    Held(const Held&) = delete;
    Held& operator=(const Held&) = delete;
    ~Held() { Py_XDECREF(o); }
    PyObject* release() {
        PyObject* const p = o;
        o = nullptr;
        return p;
    }
};

template <typename F>
PyObject* guarded(Py_ssize_t given, Py_ssize_t wanted, F&& f) {
    HANDLE_TH_ERRORS
    if (given != wanted) {
        PyErr_Format(PyExc_TypeError, "%zd arguments, not %zd", given, wanted);
        return nullptr;
    }
    try {
        return f();
    } catch (const PythonError&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// (x, perm, b, fmt, codes, scales, stream, algo, placement)
PyObject* apply(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 9, [&]() -> PyObject* {
        const Rows r = rows_of(a[0]);
        const int32_t d = (int32_t)r.d, b = (int32_t)integer(a[2]);
        const auto fmt = (perq_fmt_t)integer(a[3]);
        const auto algo = (perq_algo_t)integer(a[7]);
        if (a[8] != Py_None && algo != PERQ_ALGO_AUTO) {
            PyErr_SetString(PyExc_ValueError, "a placement goes with algo='auto'");
            throw PythonError();
        }
        const Stream stream = stream_of(a[6]);
        const bool own = a[4] == Py_None || a[5] == Py_None;
        const int64_t per_row = fmt == PERQ_FMT_MXFP4 ? r.d / 32 : 2, shape[2] = {r.T, per_row};
        const bool one = fmt != PERQ_FMT_MXFP4 && fmt != PERQ_FMT_INT4_ASYM_TOKEN;      // (asymmetric: step and zero point)
        Held codes(output(own ? Py_None : a[4], {r.T, r.d / 2}, at::kByte, r.device, stream));
        Held scales(output(own ? Py_None : a[5], at::IntArrayRef(shape, one ? 1 : 2), fmt == PERQ_FMT_MXFP4 ? at::kByte : at::kFloat, r.device, stream));
        if (a[8] != Py_None) {
            const at::Tensor& t = tensor(a[8], "placement");
            if (t.scalar_type() != at::kByte || !t.is_contiguous() || (size_t)t.numel() != perq_perm_prepared_bytes(d)) {
                PyErr_SetString(PyExc_ValueError, "placement: not the bytes perq_perm_prepare writes for rows of this width");
                throw PythonError();
            }
        }
        const auto* perm = static_cast<const int32_t*>(address(a[1]));
        const void* const placement = address(a[8]);
        auto* c = static_cast<uint8_t*>(address(codes.o));
        void* const s = address(scales.o);
        const perq_status_t st = unlocked([&] {
            return algo == PERQ_ALGO_AUTO ? perq_permute_rotate_quant_prepared(r.x, r.T, d, r.ldx, perm, placement, b, fmt, c, s, stream.raw)
                                          : perq_permute_rotate_quant_algo(r.x, r.T, d, r.ldx, perm, b, fmt, algo, c, s, stream.raw);
        });
        if (st != PERQ_OK) return PyLong_FromLong(st);
        PyObject* const both = PyTuple_New(2);
        if (both == nullptr) throw PythonError();
        PyTuple_SET_ITEM(both, 0, codes.release());
        PyTuple_SET_ITEM(both, 1, scales.release());
        return both;
    });
}

// (x, perm, b, y, stream, algo)
PyObject* rotate_f32(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 6, [&]() -> PyObject* {
        const Rows r = rows_of(a[0]);
        const int32_t b = (int32_t)integer(a[2]);
        const auto algo = (perq_algo_t)integer(a[5]);
        const Stream stream = stream_of(a[4]);
        Held y(output(a[3], {r.T, r.d}, at::kFloat, r.device, stream));
        const auto* perm = static_cast<const int32_t*>(address(a[1]));
        auto* out = static_cast<float*>(address(y.o));
        const perq_status_t st = unlocked([&] { return perq_permute_rotate_f32(r.x, r.T, (int32_t)r.d, r.ldx, perm, b, algo, out, stream.raw); });
        return result(st, y.release());
    });
}

// (x, perm, b, out, stream)
PyObject* diagnostics(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 5, [&]() -> PyObject* {
        const Rows r = rows_of(a[0]);
        const int32_t b = (int32_t)integer(a[2]);
        const Stream stream = stream_of(a[4]);
        Held out(output(a[3], {r.T, 4}, at::kFloat, r.device, stream));
        const auto* perm = static_cast<const int32_t*>(address(a[1]));
        auto* o = static_cast<float*>(address(out.o));
        const perq_status_t st = unlocked([&] { return perq_block_diagnostics(r.x, r.T, (int32_t)r.d, r.ldx, perm, b, o, stream.raw); });
        return result(st, out.release());
    });
}

// (x, out, stream, largest instead of mean)
PyObject* column_statistic(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 4, [&]() -> PyObject* {
        const Rows r = rows_of(a[0]);
        const int32_t d = (int32_t)r.d;
        const bool largest = a[3] == Py_True;
        const Stream stream = stream_of(a[2]);
        Held out(output(a[1], {r.d}, at::kFloat, r.device, stream));
        const size_t bytes = perq_colabs_mean_workspace_bytes(r.T, d);
        const at::Tensor work = buffer({(int64_t)(bytes > 16 ? bytes : 16)}, at::kByte, r.device, stream, false);
        auto* o = static_cast<float*>(address(out.o));
        void* const w = work.data_ptr();
        const perq_status_t st = unlocked([&] { return (largest ? perq_colabs_absmax : perq_colabs_mean)(r.x, r.T, d, r.ldx, o, w, bytes, stream.raw); });
        return result(st, out.release());
    });
}

// (y, codes, scales, fmt, out, stream)
PyObject* quant_error(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 6, [&]() -> PyObject* {
        const at::Tensor& y = tensor(a[0], "y");
        if (y.dim() != 2) {
            PyErr_SetString(PyExc_ValueError, "y must be a 2-D tensor");
            throw PythonError();
        }
        const int64_t T = y.size(0);
        const auto d = (int32_t)y.size(1);
        const auto fmt = (perq_fmt_t)integer(a[3]);
        const Stream stream = stream_of(a[5]);
        Held out(output(a[4], {T, 3}, at::kFloat, y.device(), stream));
        const auto* v = static_cast<const float*>(y.data_ptr());
        const auto* c = static_cast<const uint8_t*>(address(a[1]));
        const void* const s = address(a[2]);
        auto* o = static_cast<float*>(address(out.o));
        const perq_status_t st = unlocked([&] { return perq_quant_error(v, T, d, c, s, fmt, o, stream.raw); });
        return result(st, out.release());
    });
}

// (a_codes, a_scales, w_codes, w_scales, out, stream, MXFP4)
PyObject* product(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 7, [&]() -> PyObject* {
        const at::Tensor &ac = tensor(a[0], "a_codes"), &wc = tensor(a[2], "w_codes");
        const bool mx = a[6] == Py_True;
        if (ac.dim() < 2 || wc.dim() < 2 || ac.size(1) != wc.size(1) || !ac.is_contiguous() || !wc.is_contiguous()) {
            PyErr_SetString(PyExc_ValueError, "a_codes [T, d/2] and w_codes [N, d/2] must be contiguous with the same d");
            throw PythonError();
        }
        if (mx && (!tensor(a[1], "a_scales").is_contiguous() || !tensor(a[3], "w_scales").is_contiguous())) {
            PyErr_SetString(PyExc_ValueError, "scale bytes must be contiguous");
            throw PythonError();
        }
        const int64_t T = ac.size(0), N = wc.size(0);
        const auto d = (int32_t)(2 * ac.size(1));
        const Stream stream = stream_of(a[5]);
        Held out(output(a[4], {T, N}, at::kFloat, ac.device(), stream));
        const int64_t ldo = T != 0 ? tensor(out.o, "out").stride(0) : N;
        const auto *pa = static_cast<const uint8_t*>(ac.data_ptr()), *pw = static_cast<const uint8_t*>(wc.data_ptr());
        const void *const sa = address(a[1]), *const sw = address(a[3]);
        auto* o = static_cast<float*>(address(out.o));
        const perq_status_t st = unlocked([&] {
            return mx ? perq_w4a4_mxfp4_gemm_ref(pa, static_cast<const uint8_t*>(sa), T, pw, static_cast<const uint8_t*>(sw), (int32_t)N, d, o, ldo, stream.raw)
                      : perq_w4a4_gemm_ref(pa, static_cast<const float*>(sa), T, pw, static_cast<const float*>(sw), (int32_t)N, d, o, ldo, stream.raw);
        });
        return result(st, out.release());
    });
}

#define PERQ_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {PERQ_METHOD(apply), PERQ_METHOD(rotate_f32), PERQ_METHOD(diagnostics), PERQ_METHOD(column_statistic),
                         PERQ_METHOD(quant_error), PERQ_METHOD(product), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_perq_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__perq_torch(void) { return PyModule_Create(&module); }
