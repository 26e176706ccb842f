// Argument marshalling of the entry points a program calls per layer (binding.py holds the rest): torch device tensors,
// descriptors and modes in, one call of libsparq out.  The checks, their order and their messages are those the Python
// functions had; what they cost is not: five tensors' checks, the current stream and ctypes' conversions were 2.7 us of a 6.7 us call,
// of which the launch itself takes 4.  The library's functions are reached through addresses binding.py hands over, so that
// another build of the library can be loaded there.  No computation happens here and nothing is kept between calls.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "../../../include/sparq.h"

namespace {

struct Library {
    decltype(&sparq_trim) trim;
    decltype(&sparq_conv_gemm) conv_gemm;
    decltype(&sparq_conv_gemm_u8) conv_gemm_u8;
    decltype(&sparq_conv_gemm_packed) conv_gemm_packed;
    decltype(&sparq_conv_gemm_sparse24) conv_gemm_sparse24;
    decltype(&sparq_dequant) dequant;
    decltype(&sparq_requant) requant;
    decltype(&sparq_pack_act) pack_act;
    decltype(&sparq_unpack_act) unpack_act;
};
Library lib;
PyObject *mode_type, *desc_type, *error_type;        // SparqMode, SparqConvDesc, SparqError of binding.py

struct PythonError {};                               // a Python exception is set

[[noreturn]] void raise(PyObject* type, const char* text) {
    PyErr_SetString(type, text);
    throw PythonError{};
}

// ---- arguments by position and by name ----
template <int N>
struct Signature {
    const char* function;
    const char* names[N];
    int required;
    PyObject* interned[N];
};
template <int N>
void parse(Signature<N>& sig, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames, PyObject* (&out)[N]) {
    if (!sig.interned[0])
        for (int i = 0; i < N; ++i)
            if (!(sig.interned[i] = PyUnicode_InternFromString(sig.names[i]))) throw PythonError{};
    if (nargs > N) {
        PyErr_Format(PyExc_TypeError, "%s() takes at most %d positional arguments but %zd were given", sig.function, N, nargs);
        throw PythonError{};
    }
    for (int i = 0; i < N; ++i) out[i] = i < nargs ? args[i] : nullptr;
    const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < nkw; ++k) {
        PyObject* name = PyTuple_GET_ITEM(kwnames, k);
        int at = -1;
        for (int i = 0; i < N && at < 0; ++i)
            if (name == sig.interned[i]) at = i;
        for (int i = 0; i < N && at < 0; ++i)
            if (PyUnicode_Compare(name, sig.interned[i]) == 0) at = i;
        if (at < 0) {
            PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", sig.function, name);
            throw PythonError{};
        }
        if (out[at]) {
            PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%s'", sig.function, sig.names[at]);
            throw PythonError{};
        }
        out[at] = args[nargs + k];
    }
    for (int i = 0; i < sig.required; ++i)
        if (!out[i]) {
            PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", sig.function, sig.names[i]);
            throw PythonError{};
        }
}
bool given(PyObject* o) { return o && o != Py_None; }

// ---- descriptors and modes: the bytes of a ctypes structure ----
template <class T>
T structure(PyObject* o, PyObject* type, const char* what) {
    const int is = Py_TYPE(o) == reinterpret_cast<PyTypeObject*>(type) ? 1 : PyObject_IsInstance(o, type);
    if (is < 0) throw PythonError{};
    if (!is) {
        PyErr_Format(PyExc_TypeError, "expected a %s, not %s", what, Py_TYPE(o)->tp_name);
        throw PythonError{};
    }
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw PythonError{};
    T value{};
    const bool whole = view.len >= (Py_ssize_t)sizeof(T);
    if (whole) memcpy(&value, view.buf, sizeof(T));
    PyBuffer_Release(&view);
    if (!whole) raise(PyExc_TypeError, "structure too small");
    return value;
}
sparq_mode mode_of(PyObject* o) { return structure<sparq_mode>(o, mode_type, "SparqMode"); }
sparq_conv_desc desc_of(PyObject* o) { return structure<sparq_conv_desc>(o, desc_type, "SparqConvDesc"); }

// ---- tensors ----
const at::Tensor& tensor(PyObject* o, const char* name) {
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a tensor, not %s", name, Py_TYPE(o)->tp_name);
        throw PythonError{};
    }
    return THPVariable_Unpack(o);
}
template <class T>
constexpr at::ScalarType kDtype = std::is_same_v<T, uint8_t> ? at::kByte : std::is_same_v<T, int32_t> ? at::kInt : at::kFloat;
template <class T>
T* device_pointer(const at::Tensor& t, const char* name) {
    if (!t.is_cuda() || t.scalar_type() != kDtype<T> || !t.is_contiguous()) {
        PyErr_Format(PyExc_TypeError, "%s must be a contiguous device tensor of dtype %s", name,
                     kDtype<T> == at::kByte ? "torch.uint8" : kDtype<T> == at::kInt ? "torch.int32" : "torch.float32");
        throw PythonError{};
    }
    return static_cast<T*>(t.data_ptr());
}
template <class T>
T* device_pointer(PyObject* o, const char* name) { return given(o) ? device_pointer<T>(tensor(o, name), name) : nullptr; }

// The current device's current stream, as the caller sees it.
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// ---- sizes, in Python's integers ----
typedef __int128 Int;
Int floor_div(Int a, Int b) {
    if (b == 0) raise(PyExc_ZeroDivisionError, "integer division or modulo by zero");
    const Int q = a / b;
    return q * b != a && (a < 0) != (b < 0) ? q - 1 : q;
}
Int out_rows(const sparq_conv_desc& d) {
    return d.B * (floor_div((Int)d.H + 2 * (Int)d.pad_h - d.KH, d.stride_h) + 1) * (floor_div((Int)d.W + 2 * (Int)d.pad_w - d.KW, d.stride_w) + 1);
}
void check_input(PyObject* x, const sparq_conv_desc& d) {
    if (tensor(x, "x").numel() != (Int)d.B * d.H * d.W * d.C) raise(PyExc_ValueError, "activation size does not match the descriptor");
}
void check_results(PyObject* t, const char* name, Int elements) {
    if (!given(t) || tensor(t, name).numel() == elements) return;
    PyErr_Format(PyExc_ValueError, "%s must hold M*N = %lld elements", name, (long long)elements);
    throw PythonError{};
}
void check_channels(PyObject* t, const char* name, int n) {
    if (!given(t) || tensor(t, name).numel() == n) return;
    PyErr_Format(PyExc_ValueError, "%s must hold N elements", name);
    throw PythonError{};
}
int64_t last_axis(const at::Tensor& t) {
    if (t.dim() == 0) raise(PyExc_IndexError, "tuple index out of range");
    return t.size(t.dim() - 1);
}
int64_t rows_of(const at::Tensor& t, int64_t channels) { return (int64_t)floor_div(t.numel(), channels); }
int32_t group_of(PyObject* o) {
    if (!o) return 1;
    PyObject* n = PyNumber_Long(o);
    if (!n) throw PythonError{};
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    if (PyErr_Occurred()) throw PythonError{};
    return (int32_t)v;
}

// ---- one call of the library, other Python threads running ----
template <class F>
PyObject* call(const char* what, F&& f) {
    PyThreadState* state = PyEval_SaveThread();
    const sparq_status status = f();
    PyEval_RestoreThread(state);
    if (status == SPARQ_OK) Py_RETURN_NONE;
    PyObject* e = PyObject_CallFunction(error_type, "is", (int)status, what);
    if (e) {
        PyErr_SetObject(error_type, e);
        Py_DECREF(e);
    }
    throw PythonError{};
}
template <PyObject* (*F)(PyObject* const*, Py_ssize_t, PyObject*)>
PyObject* guarded(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    try {
        return F(args, nargs, kwnames);
    } catch (const PythonError&) {
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "unknown error");
    }
    return nullptr;
}

PyObject* conv_gemm(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static Signature<8> sig = {"sparq_conv_gemm", {"x", "packed", "d", "m", "acc", "scale", "out", "workspace"}, 4, {}};
    PyObject* a[8];
    parse(sig, args, nargs, kwnames, a);
    const sparq_conv_desc d = desc_of(a[2]);
    check_input(a[0], d);
    const Int elements = out_rows(d) * d.N;
    check_results(a[4], "acc", elements);
    check_results(a[6], "out", elements);
    check_channels(a[5], "scale", d.N);
    uint8_t* ws = device_pointer<uint8_t>(a[7], "workspace");
    const size_t ws_bytes = given(a[7]) ? (size_t)tensor(a[7], "workspace").numel() : 0;
    const uint8_t *x = device_pointer<uint8_t>(a[0], "x"), *packed = device_pointer<uint8_t>(a[1], "packed");
    const sparq_mode m = mode_of(a[3]);
    int32_t* acc = device_pointer<int32_t>(a[4], "acc");
    const float* scale = device_pointer<float>(a[5], "scale");
    float* out = device_pointer<float>(a[6], "out");
    void* s = stream();
    return call("sparq_conv_gemm", [&] { return lib.conv_gemm(x, packed, &d, &m, acc, scale, out, ws, ws_bytes, s); });
}

PyObject* conv_gemm_u8(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static Signature<8> sig = {"sparq_conv_gemm_u8", {"x", "packed", "d", "m", "factor", "y", "workspace", "out_mode"}, 6, {}};
    PyObject* a[8];
    parse(sig, args, nargs, kwnames, a);
    const sparq_conv_desc d = desc_of(a[2]);
    check_input(a[0], d);
    const Int elements = out_rows(d) * d.N;
    if (tensor(a[5], "y").numel() != elements) check_results(a[5], "y", elements);
    if (tensor(a[4], "factor").numel() != d.N) check_channels(a[4], "factor", d.N);
    uint8_t* ws = device_pointer<uint8_t>(a[6], "workspace");
    const size_t ws_bytes = given(a[6]) ? (size_t)tensor(a[6], "workspace").numel() : 0;
    const uint8_t *x = device_pointer<uint8_t>(a[0], "x"), *packed = device_pointer<uint8_t>(a[1], "packed");
    const sparq_mode m = mode_of(a[3]);
    const float* factor = device_pointer<float>(a[4], "factor");
    uint8_t* y = device_pointer<uint8_t>(a[5], "y");
    const bool trims = given(a[7]);
    const sparq_mode om = trims ? mode_of(a[7]) : sparq_mode{};
    void* s = stream();
    return call("sparq_conv_gemm_u8",
                [&] { return lib.conv_gemm_u8(x, packed, &d, &m, factor, y, trims ? &om : nullptr, ws, ws_bytes, s); });
}

PyObject* conv_gemm_packed(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static Signature<9> sig = {"sparq_conv_gemm_packed", {"packed_x", "group", "packed_w", "d", "m", "acc", "scale", "out", "workspace"}, 5, {}};
    PyObject* a[9];
    parse(sig, args, nargs, kwnames, a);
    const sparq_conv_desc d = desc_of(a[3]);
    const Int elements = out_rows(d) * d.N;
    check_results(a[5], "acc", elements);
    check_results(a[7], "out", elements);
    check_channels(a[6], "scale", d.N);
    uint8_t* ws = device_pointer<uint8_t>(a[8], "workspace");
    const size_t ws_bytes = given(a[8]) ? (size_t)tensor(a[8], "workspace").numel() : 0;
    const at::Tensor& px = tensor(a[0], "packed_x");
    const uint8_t* x = device_pointer<uint8_t>(px, "packed_x");
    const size_t x_bytes = (size_t)px.numel();
    const int32_t group = group_of(a[1]);
    const uint8_t* packed = device_pointer<uint8_t>(a[2], "packed_w");
    const sparq_mode m = mode_of(a[4]);
    int32_t* acc = device_pointer<int32_t>(a[5], "acc");
    const float* scale = device_pointer<float>(a[6], "scale");
    float* out = device_pointer<float>(a[7], "out");
    void* s = stream();
    return call("sparq_conv_gemm_packed",
                [&] { return lib.conv_gemm_packed(x, x_bytes, group, packed, &d, &m, acc, scale, out, ws, ws_bytes, s); });
}

PyObject* conv_gemm_sparse24(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static Signature<8> sig = {"sparq_conv_gemm_sparse24", {"x", "packed", "d", "m", "acc", "scale", "out", "workspace"}, 4, {}};
    PyObject* a[8];
    parse(sig, args, nargs, kwnames, a);
    const sparq_conv_desc d = desc_of(a[2]);
    check_input(a[0], d);
    const Int elements = out_rows(d) * d.N;
    check_results(a[4], "acc", elements);
    check_results(a[6], "out", elements);
    uint8_t* ws = device_pointer<uint8_t>(a[7], "workspace");
    const size_t ws_bytes = given(a[7]) ? (size_t)tensor(a[7], "workspace").numel() : 0;
    const uint8_t *x = device_pointer<uint8_t>(a[0], "x"), *packed = device_pointer<uint8_t>(a[1], "packed");
    const sparq_mode m = mode_of(a[3]);
    int32_t* acc = device_pointer<int32_t>(a[4], "acc");
    const float* scale = device_pointer<float>(a[5], "scale");
    float* out = device_pointer<float>(a[6], "out");
    void* s = stream();
    return call("sparq_conv_gemm_sparse24", [&] { return lib.conv_gemm_sparse24(x, packed, &d, &m, acc, scale, out, ws, ws_bytes, s); });
}

PyObject* trim(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static Signature<3> sig = {"sparq_trim", {"x", "y", "m"}, 3, {}};
    PyObject* a[3];
    parse(sig, args, nargs, kwnames, a);
    const at::Tensor &x = tensor(a[0], "x"), &y = tensor(a[1], "y");
    const int64_t channels = last_axis(x), rows = channels ? x.numel() / channels : 0;
    if (x.sizes() != y.sizes()) raise(PyExc_ValueError, "x and y must have the same shape");
    const uint8_t* xp = device_pointer<uint8_t>(x, "x");
    uint8_t* yp = device_pointer<uint8_t>(y, "y");
    const sparq_mode m = mode_of(a[2]);
    void* s = stream();
    return call("sparq_trim", [&] { return lib.trim(xp, yp, rows, (int32_t)channels, &m, s); });
}

// acc [M][N], one factor per column, results of acc's shape
template <class Out, class F>
PyObject* per_channel(const char* what, PyObject* const (&a)[3], const char* factor_name, const char* out_name, F&& f) {
    const at::Tensor &acc = tensor(a[0], "acc"), &factor = tensor(a[1], factor_name), &out = tensor(a[2], out_name);
    if (acc.dim() != 2) raise(PyExc_ValueError, "acc must have two dimensions");
    const int64_t rows = acc.size(0), n = acc.size(1);
    if (out.sizes() != acc.sizes() || factor.numel() != n) raise(PyExc_ValueError, "shape mismatch");
    const int32_t* ap = device_pointer<int32_t>(acc, "acc");
    const float* fp = device_pointer<float>(factor, factor_name);
    Out* op = device_pointer<Out>(out, out_name);
    void* s = stream();
    return call(what, [&] { return f(ap, fp, op, rows, (int32_t)n, s); });
}
PyObject* dequant(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static Signature<3> sig = {"sparq_dequant", {"acc", "scale", "out"}, 3, {}};
    PyObject* a[3];
    parse(sig, args, nargs, kwnames, a);
    return per_channel<float>("sparq_dequant", a, "scale", "out", lib.dequant);
}
PyObject* requant(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static Signature<3> sig = {"sparq_requant", {"acc", "factor", "y"}, 3, {}};
    PyObject* a[3];
    parse(sig, args, nargs, kwnames, a);
    return per_channel<uint8_t>("sparq_requant", a, "factor", "y", lib.requant);
}

PyObject* pack_act(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static Signature<4> sig = {"sparq_pack_act", {"x", "packed", "m", "group"}, 3, {}};
    PyObject* a[4];
    parse(sig, args, nargs, kwnames, a);
    const at::Tensor &x = tensor(a[0], "x"), &packed = tensor(a[1], "packed");
    const int64_t channels = last_axis(x);
    const uint8_t* xp = device_pointer<uint8_t>(x, "x");
    uint8_t* pp = device_pointer<uint8_t>(packed, "packed");
    const int64_t bytes = packed.numel(), rows = rows_of(x, channels);
    const sparq_mode m = mode_of(a[2]);
    const int32_t group = group_of(a[3]);
    void* s = stream();
    return call("sparq_pack_act", [&] { return lib.pack_act(xp, pp, (size_t)bytes, rows, (int32_t)channels, &m, group, s); });
}
PyObject* unpack_act(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static Signature<4> sig = {"sparq_unpack_act", {"packed", "y", "m", "group"}, 3, {}};
    PyObject* a[4];
    parse(sig, args, nargs, kwnames, a);
    const at::Tensor &packed = tensor(a[0], "packed"), &y = tensor(a[1], "y");
    const int64_t channels = last_axis(y);
    const uint8_t* pp = device_pointer<uint8_t>(packed, "packed");
    const int64_t bytes = packed.numel();
    uint8_t* yp = device_pointer<uint8_t>(y, "y");
    const int64_t rows = rows_of(y, channels);
    const sparq_mode m = mode_of(a[2]);
    const int32_t group = group_of(a[3]);
    void* s = stream();
    return call("sparq_unpack_act", [&] { return lib.unpack_act(pp, (size_t)bytes, yp, rows, (int32_t)channels, &m, group, s); });
}

// bind(addresses, SparqMode, SparqConvDesc, SparqError): addresses of the library's functions, in Library's order
PyObject* bind(PyObject*, PyObject* args) {
    PyObject* list;
    if (!PyArg_ParseTuple(args, "O!OOO", &PyTuple_Type, &list, &mode_type, &desc_type, &error_type)) return nullptr;
    constexpr Py_ssize_t n = sizeof(Library) / sizeof(void*);
    if (PyTuple_GET_SIZE(list) != n) {
        PyErr_SetString(PyExc_ValueError, "one address per function");
        return nullptr;
    }
    void* addresses[n];
    for (Py_ssize_t i = 0; i < n; ++i) {
        addresses[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(list, i));
        if (PyErr_Occurred()) return nullptr;
    }
    memcpy(&lib, addresses, sizeof(lib));
    Py_INCREF(mode_type);
    Py_INCREF(desc_type);
    Py_INCREF(error_type);
    Py_RETURN_NONE;
}

#define SPARQ_METHOD(F, DOC) \
    {"sparq_" #F, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(guarded<F>)), METH_FASTCALL | METH_KEYWORDS, "sparq_" #F DOC}
PyMethodDef methods[] = {
    SPARQ_METHOD(trim, "(x, y, m)\n--\n\ny = vSPARQ/bSPARQ-trimmed x along the last axis (uint8 device tensors; y may be x)."),
    SPARQ_METHOD(conv_gemm, "(x, packed, d, m, acc=None, scale=None, out=None, workspace=None)\n--\n\n"
                            "The trimmed convolution: acc = int32 sums, out = acc * scale per output channel."),
    SPARQ_METHOD(conv_gemm_u8, "(x, packed, d, m, factor, y, workspace=None, out_mode=None)\n--\n\n"
                               "The convolution with its result requantised to uint8 (y holds M*N bytes: the next layer's NHWC input), "
                               "optionally trimmed with out_mode as the next layer would trim it on loading."),
    SPARQ_METHOD(conv_gemm_packed, "(packed_x, group, packed_w, d, m, acc=None, scale=None, out=None, workspace=None)\n--\n\n"
                                   "sparq_conv_gemm on an input held in packed storage (written by sparq_pack_act with the same mode and group)."),
    SPARQ_METHOD(conv_gemm_sparse24, "(x, packed, d, m, acc=None, scale=None, out=None, workspace=None)\n--\n\n"
                                     "The convolution with 2:4 pruned weights: activations picked by the weights' coordinates, then paired."),
    SPARQ_METHOD(dequant, "(acc, scale, out)\n--\n\nout = float(acc) * scale[n] for acc [M][N]."),
    SPARQ_METHOD(requant, "(acc, factor, y)\n--\n\ny = clamp(round(acc * factor[n]), 0, 255) for acc [M][N]."),
    SPARQ_METHOD(pack_act, "(x, packed, m, group=1)\n--\n\n"
                           "packed (uint8 device buffer) = the n-bit data + ShiftCtrl + MuxCtrl records of the trimmed x (last axis = channels)."),
    SPARQ_METHOD(unpack_act, "(packed, y, m, group=1)\n--\n\ny (uint8, last axis = channels) = the values the records encode."),
    {"bind", bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_sparq_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__sparq_native() { return PyModule_Create(&module_def); }
