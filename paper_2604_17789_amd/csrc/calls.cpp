// The binding's calls for serving and analysis with the work between Python and the C ABI (include/duqpp.h) in native code.
//
// A call through ctypes costs the host about 5 us beside its launches (2.3 us each): attributes of half a dozen tensors read one
// by one from Python and sixteen arguments converted.  Here they are read from the tensors themselves.
// Per call with its buffers given, two launches: 9.1 -> 5.5 us.
//
// Each function does the plain case and nothing else: tensors of the expected types, layouts and sizes, Python integers, no
// torch function or dispatch mode in force.  For everything else, and for whatever throws, it answers None, and the Python code
// that called it goes on with its own checks, which refuse and accept as they always have.  Nothing has been launched then, but
// where the wait in error() throws.  Otherwise the result, or the C call's status as an int where that is not 0.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/autograd/python_variable.h>

#include "duqpp.h"

namespace {

constexpr int64_t kMost = (int64_t)1 << 30;              // rows and K the library takes

decltype(&duqpp_rotq_gemm_tiled_packed) rotq_gemm_tiled_packed;
decltype(&duqpp_rotq_gemm_tiled) rotq_gemm_tiled;
decltype(&duqpp_rotq_gemm) rotq_gemm;
decltype(&duqpp_gemm_workspace_bytes) gemm_workspace_bytes;
decltype(&duqpp_rotate_quantize_tiled_packed) rotate_quantize_tiled_packed;
decltype(&duqpp_rotate_quantize_tiled) rotate_quantize_tiled;
decltype(&duqpp_quantize_weights_tiled) quantize_weights_tiled;
decltype(&duqpp_mxfp4_gemm_tiled) mxfp4_gemm_tiled;
decltype(&duqpp_group_error_partials) group_error_partials;
decltype(&duqpp_group_error_partials_bytes) group_error_partials_bytes;
decltype(&duqpp_group_error_mean) group_error_mean;
PyObject* current_stream;                                // the binding's function that answers it as an integer

// The Python threads run while the object lives.
struct WithoutGil {
    PyThreadState* state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

bool plain_torch() {
    return !at::impl::torch_function_mode_enabled() && c10::impl::TorchDispatchModeTLS::stack_len() == 0 &&
           !c10::impl::TorchDispatchModeTLS::any_modes_set();
}

// The tensor of a Python object, null where it is none of torch's own type on the GPU.
const at::Tensor* tensor(PyObject* o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.scalar_type() == type && t.layout() == at::kStrided ? &t : nullptr;
}
// bytes that the library reads or writes as one run
const at::Tensor* bytes(PyObject* o) {
    const at::Tensor* t = tensor(o, at::kByte);
    return t && t->is_contiguous() ? t : nullptr;
}
const at::Tensor* matrix(PyObject* o, at::ScalarType type) {
    const at::Tensor* t = tensor(o, type);
    return t && t->dim() == 2 && t->stride(1) == 1 ? t : nullptr;
}
const at::Tensor* blocks(PyObject* o) {
    const at::Tensor* t = tensor(o, at::kFloat);
    return t && t->dim() == 3 && t->size(1) == 32 && t->size(2) == 32 && t->is_contiguous() ? t : nullptr;
}
constexpr int64_t kPackedBlock = 6144;
const at::Tensor* packed_blocks(PyObject* o) {
    const at::Tensor* t = bytes(o);
    return t && t->dim() == 1 && t->numel() > 0 && t->numel() % kPackedBlock == 0 ? t : nullptr;
}
bool integer(PyObject* o, long long& v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
// out_dtype as the C call takes it
bool result_type(PyObject* o, long long& code, at::ScalarType& type) {
    if (!integer(o, code) || (code != DUQPP_F32 && code != DUQPP_BF16)) return false;
    type = code == DUQPP_F32 ? at::kFloat : at::kBFloat16;
    return true;
}
// the current stream of the current device; false: the binding's function threw
bool stream_of_call(void*& stream) {
    PyObject* o = PyObject_CallNoArgs(current_stream);
    stream = o ? PyLong_AsVoidPtr(o) : nullptr;
    Py_XDECREF(o);
    if (!PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}

bool sizes_ok(int64_t rows, int64_t K) { return rows >= 1 && rows <= kMost && K >= 32 && K <= kMost && K % 32 == 0; }
int64_t tiled_units(int64_t rows, int64_t K) { return (rows + 31) / 32 * ((K + 255) / 256); }   // 4096 code and 256 scale bytes each

at::Tensor device_empty(at::IntArrayRef sizes, at::ScalarType type, const at::Tensor& like) {
    return at::empty(sizes, at::TensorOptions().dtype(type).device(like.device()));
}

// `out` as given, or undefined where it is None (allocated once the interpreter is let go); false: neither.
bool given_result(PyObject* o, int64_t T, int64_t N, at::ScalarType type, at::Tensor& y) {
    if (o == Py_None) return true;
    const at::Tensor* t = matrix(o, type);
    if (!t || t->size(0) != T || t->size(1) != N) return false;
    y = *t;
    return true;
}

template <typename F>
PyObject* guarded(F&& f) {
    try {
        if (!plain_torch()) Py_RETURN_NONE;
        return f();
    } catch (...) {                                          // the Python path meets the same, and says so
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

enum Linear { kPacked = 0, kBlocks = 1, kRowMajor = 2 };

// linear(form, x, R, b_codes, b_scales, N, out_dtype, out, workspace) -> y
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        long long form, N = 0, code;
        at::ScalarType type;
        void* stream;
        if (n != 9 || !integer(a[0], form) || !result_type(a[6], code, type)) Py_RETURN_NONE;
        const at::Tensor* x = matrix(a[1], at::kBFloat16);
        const at::Tensor* R = form == kPacked ? packed_blocks(a[2]) : blocks(a[2]);
        const at::Tensor *bc = bytes(a[3]), *bs = bytes(a[4]);
        if (!x || !R || !bc || !bs) Py_RETURN_NONE;
        const int64_t T = x->size(0), K = x->size(1);
        if (form == kRowMajor) {
            if (bc->dim() != 2 || bs->dim() != 2) Py_RETURN_NONE;
            N = bc->size(0);
            if (!sizes_ok(T, K) || !sizes_ok(N, K) || bc->size(1) * 2 != K || bs->size(0) != N || bs->size(1) != K / 32) Py_RETURN_NONE;
        } else if (!integer(a[5], N) || !sizes_ok(T, K) || !sizes_ok(N, K) || bc->numel() != tiled_units(N, K) * 4096 ||
                   bs->numel() != tiled_units(N, K) * 256) {
            Py_RETURN_NONE;
        }
        const int64_t nb = form == kPacked ? R->numel() / kPackedBlock : R->size(0);
        at::Tensor y, ws;
        if (!given_result(a[7], T, N, type, y)) Py_RETURN_NONE;
        if (a[8] != Py_None) {
            const at::Tensor* t = bytes(a[8]);
            if (!t) Py_RETURN_NONE;
            ws = *t;
        }
        if (!stream_of_call(stream)) Py_RETURN_NONE;
        int status;
        {
            WithoutGil threads;
            if (!y.defined()) y = device_empty({T, N}, type, *x);
            if (!ws.defined())
                ws = device_empty({form == kRowMajor ? (int64_t)gemm_workspace_bytes(T, N, K, 1) : tiled_units(T, K) * 4352}, at::kByte, *x);
            const uint8_t *bcp = static_cast<const uint8_t*>(bc->data_ptr()), *bsp = static_cast<const uint8_t*>(bs->data_ptr());
            void* w = ws.data_ptr();
            const size_t wn = (size_t)ws.numel();
            if (form == kPacked)
                status = rotq_gemm_tiled_packed(x->data_ptr(), x->stride(0), R->data_ptr(), nb, bcp, bsp, T, N, K, y.data_ptr(), (int)code,
                                                y.stride(0), w, wn, stream);
            else if (form == kBlocks)
                status = rotq_gemm_tiled(x->data_ptr(), x->stride(0), static_cast<const float*>(R->data_ptr()), nb, bcp, bsp, T, N, K,
                                         y.data_ptr(), (int)code, y.stride(0), w, wn, stream);
            else
                status = rotq_gemm(x->data_ptr(), x->stride(0), static_cast<const float*>(R->data_ptr()), nb, bcp, bsp, T, N, K, y.data_ptr(),
                                   (int)code, y.stride(0), w, wn, stream);
        }
        if (status != DUQPP_OK) return PyLong_FromLong(status);
        if (a[7] != Py_None) {
            Py_INCREF(a[7]);
            return a[7];
        }
        return THPVariable_Wrap(std::move(y));
    });
}

enum Rows { kRotatePacked = 0, kRotate = 1, kWeights = 2 };

// rows(form, x, R, out) -> (codes_t, scales_t)
PyObject* rows(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        long long form;
        void* stream;
        if (n != 4 || !integer(a[0], form)) Py_RETURN_NONE;
        const at::Tensor* x = matrix(a[1], at::kBFloat16);
        const at::Tensor* R = form == kRotatePacked ? packed_blocks(a[2]) : blocks(a[2]);
        if (!x || !R || !sizes_ok(x->size(0), x->size(1))) Py_RETURN_NONE;
        const int64_t T = x->size(0), K = x->size(1), units = tiled_units(T, K);
        const int64_t nb = form == kRotatePacked ? R->numel() / kPackedBlock : R->size(0);
        at::Tensor c, s;
        if (a[3] != Py_None) {
            if (!PyTuple_CheckExact(a[3]) || PyTuple_GET_SIZE(a[3]) != 2) Py_RETURN_NONE;
            const at::Tensor *gc = bytes(PyTuple_GET_ITEM(a[3], 0)), *gs = bytes(PyTuple_GET_ITEM(a[3], 1));
            if (!gc || !gs || gc->numel() != units * 4096 || gs->numel() != units * 256) Py_RETURN_NONE;
            c = *gc;
            s = *gs;
        }
        if (!stream_of_call(stream)) Py_RETURN_NONE;
        int status;
        {
            WithoutGil threads;
            if (!c.defined()) {
                c = device_empty({units * 4096}, at::kByte, *x);
                s = device_empty({units * 256}, at::kByte, *x);
            }
            uint8_t *cp = static_cast<uint8_t*>(c.data_ptr()), *sp = static_cast<uint8_t*>(s.data_ptr());
            status = form == kRotatePacked ? rotate_quantize_tiled_packed(x->data_ptr(), T, K, x->stride(0), R->data_ptr(), nb, cp, sp, stream)
                                           : (form == kRotate ? rotate_quantize_tiled : quantize_weights_tiled)(
                                                 x->data_ptr(), T, K, x->stride(0), static_cast<const float*>(R->data_ptr()), nb, cp, sp, stream);
        }
        if (status != DUQPP_OK) return PyLong_FromLong(status);
        if (a[3] != Py_None) {
            return PyTuple_Pack(2, PyTuple_GET_ITEM(a[3], 0), PyTuple_GET_ITEM(a[3], 1));
        }
        PyObject *co = THPVariable_Wrap(std::move(c)), *so = THPVariable_Wrap(std::move(s));
        PyObject* both = co && so ? PyTuple_Pack(2, co, so) : nullptr;
        Py_XDECREF(co);
        Py_XDECREF(so);
        return both;
    });
}

// product(a_codes_t, a_scales_t, b_codes_t, b_scales_t, T, N, K, out_dtype, out) -> y
PyObject* product(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        long long T, N, K, code;
        at::ScalarType type;
        void* stream;
        if (n != 9 || !integer(a[4], T) || !integer(a[5], N) || !integer(a[6], K) || !result_type(a[7], code, type) || !sizes_ok(T, K) ||
            !sizes_ok(N, K))
            Py_RETURN_NONE;
        const at::Tensor* t[4];
        for (int i = 0; i < 4; ++i) {
            t[i] = bytes(a[i]);
            if (!t[i] || t[i]->numel() != tiled_units(i < 2 ? T : N, K) * (i % 2 ? 256 : 4096)) Py_RETURN_NONE;
        }
        at::Tensor y;
        if (!given_result(a[8], T, N, type, y) || !stream_of_call(stream)) Py_RETURN_NONE;
        int status;
        {
            WithoutGil threads;
            if (!y.defined()) y = device_empty({T, N}, type, *t[0]);
            const uint8_t* p[4];
            for (int i = 0; i < 4; ++i) p[i] = static_cast<const uint8_t*>(t[i]->data_ptr());
            status = mxfp4_gemm_tiled(p[0], p[1], p[2], p[3], T, N, K, y.data_ptr(), (int)code, y.stride(0), stream);
        }
        if (status != DUQPP_OK) return PyLong_FromLong(status);
        if (a[8] != Py_None) {
            Py_INCREF(a[8]);
            return a[8];
        }
        return THPVariable_Wrap(std::move(y));
    });
}

// error(x, R or None) -> (err, mean): what the mean is formed from comes by host memory that the kernel writes, one wait for the
// stream instead of another launch, a copy back and its own.
PyObject* error(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        void* stream;
        if (n != 2) Py_RETURN_NONE;
        const at::Tensor *x = matrix(a[0], at::kBFloat16), *R = nullptr;
        if (!x || !sizes_ok(x->size(0), x->size(1))) Py_RETURN_NONE;
        if (a[1] != Py_None && !(R = blocks(a[1]))) Py_RETURN_NONE;
        const int64_t T = x->size(0), K = x->size(1);
        const size_t bytes = group_error_partials_bytes(T, K);
        if (bytes == 0 || bytes > 65536 || !stream_of_call(stream)) Py_RETURN_NONE;
        at::Tensor err;
        double mean = 0.0;
        int status;
        {
            WithoutGil threads;
            err = device_empty({T, K / 32}, at::kFloat, *x);
            const at::Tensor m = at::empty({(int64_t)bytes / 8}, at::TensorOptions().dtype(at::kDouble).pinned_memory(true));
            double* const partials = static_cast<double*>(m.data_ptr());
            status = group_error_partials(x->data_ptr(), T, K, x->stride(0), R ? static_cast<const float*>(R->data_ptr()) : nullptr,
                                          R ? R->size(0) : 1, static_cast<float*>(err.data_ptr()), partials, bytes, stream);
            if (status == DUQPP_OK) {
                const c10::impl::VirtualGuardImpl device(c10::DeviceType::CUDA);
                device.synchronizeStream(device.getStream(device.getDevice()));
                mean = group_error_mean(partials, bytes);
            }
        }
        if (status != DUQPP_OK) return PyLong_FromLong(status);
        PyObject* eo = THPVariable_Wrap(std::move(err));
        PyObject* mo = PyFloat_FromDouble(mean);
        PyObject* both = eo && mo ? PyTuple_Pack(2, eo, mo) : nullptr;
        Py_XDECREF(eo);
        Py_XDECREF(mo);
        return both;
    });
}

// bind({name: address}, current stream): the C ABI's functions, from the library that the binding has loaded.
PyObject* bind(PyObject*, PyObject* args) {
    PyObject *names, *stream;
    if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &names, &stream)) return nullptr;
    auto take = [&](const char* name, auto& f) {
        PyObject* o = PyDict_GetItemString(names, name);
        void* p = o ? PyLong_AsVoidPtr(o) : nullptr;
        if (!p && !PyErr_Occurred()) PyErr_Format(PyExc_ImportError, "no address of %s", name);
        f = reinterpret_cast<std::remove_reference_t<decltype(f)>>(p);
        return p != nullptr;
    };
    if (!take("duqpp_rotq_gemm_tiled_packed", rotq_gemm_tiled_packed) || !take("duqpp_rotq_gemm_tiled", rotq_gemm_tiled) ||
        !take("duqpp_rotq_gemm", rotq_gemm) || !take("duqpp_gemm_workspace_bytes", gemm_workspace_bytes) ||
        !take("duqpp_rotate_quantize_tiled_packed", rotate_quantize_tiled_packed) ||
        !take("duqpp_rotate_quantize_tiled", rotate_quantize_tiled) || !take("duqpp_quantize_weights_tiled", quantize_weights_tiled) ||
        !take("duqpp_mxfp4_gemm_tiled", mxfp4_gemm_tiled) || !take("duqpp_group_error_partials", group_error_partials) ||
        !take("duqpp_group_error_partials_bytes", group_error_partials_bytes) || !take("duqpp_group_error_mean", group_error_mean))
        return nullptr;
    Py_INCREF(stream);
    Py_XSETREF(current_stream, stream);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(linear)), METH_FASTCALL, nullptr},
    {"rows", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(rows)), METH_FASTCALL, nullptr},
    {"product", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(product)), METH_FASTCALL, nullptr},
    {"error", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(error)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

#define TEXT_OF(x) #x
#define TEXT(x) TEXT_OF(x)

// built_for: what the binding compares with what runs, since torch's classes are read here by the layout they were compiled with.
PyMODINIT_FUNC PyInit__calls() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", "torch " DUQPP_BUILT_WITH_TORCH ", Python " TEXT(PY_MAJOR_VERSION) "." TEXT(PY_MINOR_VERSION)) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
