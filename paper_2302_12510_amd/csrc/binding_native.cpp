// Argument marshalling of binding.py in native code: the C entry points that launch work as Python functions that take
// tensors, (bits, signed) pairs, numbers and a stream in the order of their prototypes and return the status.
//
// A call through ctypes cost 6 to 7 us of argument conversion (a structure per format, a wrapper per pointer, the stream
// object), more than most small kernels run for: scale, encode and product of 64 x 64 x 256 took 26.8 us, 16.6 us with this
// module; a quantizer step on 2.4 M weights 28.9 -> 20.4 us.  The conversions are derived from the prototypes in
// dybit.h; what the arguments have to satisfy (device memory, contiguity) is checked as before.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ops/empty.h>
#include <c10/core/Allocator.h>
#include <c10/hip/HIPStream.h>
#include <c10/util/Exception.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/dybit.h"

namespace {

// A Python error is set; travels to the wrapper, which returns NULL.
struct PythonError {};

int64_t integer(PyObject *o)
{
    PyObject *i = PyNumber_Index(o);
    if (!i) throw PythonError();
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(i);      // as ctypes: reduced to the parameter's width
    Py_DECREF(i);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) throw PythonError();
    return (int64_t)v;
}

bool truth(PyObject *o)
{
    const int t = PyObject_IsTrue(o);
    if (t < 0) throw PythonError();
    return t != 0;
}

bool is_plain_tensor(PyObject *o) { return THPVariable_CheckExact(o) || Py_TYPE(o) == (PyTypeObject *)ParameterClass; }

// The address behind a tensor argument; None is NULL.
void *address(PyObject *o)
{
    if (o == Py_None) return nullptr;
    if (is_plain_tensor(o)) {
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.is_cuda()) { PyErr_SetString(PyExc_ValueError, "expected a device tensor"); throw PythonError(); }
        if (!t.is_contiguous()) { PyErr_SetString(PyExc_ValueError, "expected a contiguous tensor"); throw PythonError(); }
        return t.data_ptr();
    }
    // anything else that behaves like a tensor (subclasses) speaks for itself
    auto owned = [](PyObject *r) { if (!r) throw PythonError(); return r; };
    PyObject *r = owned(PyObject_GetAttrString(o, "is_cuda"));
    const bool cuda = PyObject_IsTrue(r) == 1;
    Py_DECREF(r);
    if (!cuda) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "expected a device tensor"); throw PythonError(); }
    r = owned(PyObject_CallMethod(o, "is_contiguous", nullptr));
    const bool contiguous = PyObject_IsTrue(r) == 1;
    Py_DECREF(r);
    if (!contiguous) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "expected a contiguous tensor"); throw PythonError(); }
    r = owned(PyObject_CallMethod(o, "data_ptr", nullptr));
    const unsigned long long p = PyLong_AsUnsignedLongLong(r);
    Py_DECREF(r);
    if (PyErr_Occurred()) throw PythonError();
    return (void *)p;
}

// None: the current stream; else a torch stream.
dybit_stream stream_of(PyObject *o)
{
    if (o == Py_None) return (dybit_stream)c10::hip::getCurrentHIPStream().stream();
    PyObject *s = PyObject_GetAttrString(o, "cuda_stream");
    if (!s) throw PythonError();
    const unsigned long long v = PyLong_AsUnsignedLongLong(s);
    Py_DECREF(s);
    if (PyErr_Occurred()) throw PythonError();
    return (dybit_stream)v;
}

dybit_fmt format(PyObject *o)
{
    PyObject *pair = PySequence_Fast(o, "expected a (bits, signed) pair");
    if (!pair) throw PythonError();
    dybit_fmt f{0, 0};
    bool ok = PySequence_Fast_GET_SIZE(pair) == 2;
    if (!ok) PyErr_SetString(PyExc_TypeError, "expected a (bits, signed) pair");
    if (ok) {
        PyObject *bits = PyNumber_Long(PySequence_Fast_GET_ITEM(pair, 0));
        const int s = PyObject_IsTrue(PySequence_Fast_GET_ITEM(pair, 1));
        ok = bits && s >= 0;
        if (bits) f.bits = (int32_t)PyLong_AsUnsignedLongLongMask(bits);
        f.is_signed = s > 0;
        Py_XDECREF(bits);
    }
    Py_DECREF(pair);
    if (!ok || PyErr_Occurred()) throw PythonError();
    return f;
}

template <class T> T argument(PyObject *o)
{
    if constexpr (std::is_same_v<T, dybit_fmt>) return format(o);
    else if constexpr (std::is_same_v<T, dybit_stream>) return stream_of(o);
    else if constexpr (std::is_pointer_v<T>) return (T)address(o);
    else { static_assert(std::is_integral_v<T>); return PyBool_Check(o) ? (T)(o == Py_True) : (T)integer(o); }
}

template <auto F> struct Entry;
template <class... A, dybit_status (*F)(A...)> struct Entry<F> {
    static constexpr Py_ssize_t kCount = sizeof...(A);
    using Arguments = std::tuple<A...>;
    template <size_t... I>
    static Arguments convert(PyObject *const *args, std::index_sequence<I...>) { return Arguments{argument<A>(args[I])...}; }   // braces: left to right
    static Arguments arguments(PyObject *const *args) { return convert(args, std::index_sequence_for<A...>{}); }
    static dybit_status run(const Arguments &a)
    {
        dybit_status st;
        Py_BEGIN_ALLOW_THREADS
        st = std::apply(F, a);
        Py_END_ALLOW_THREADS
        return st;
    }
    static PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n)
    {
        HANDLE_TH_ERRORS
        if (n != kCount) {
            PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", kCount, n);
            return nullptr;
        }
        try {
            return PyLong_FromLong((long)run(arguments(args)));
        } catch (const PythonError &) {
            return nullptr;
        }
        END_HANDLE_TH_ERRORS
    }
};

// Memory of the current device that later work on its current stream may reuse once the result is gone; empty where there is not enough:
// what is only faster with a workspace does without one then.
c10::DataPtr scratch(size_t bytes)
{
    try {
        return c10::GetAllocator(c10::DeviceType::CUDA)->allocate(bytes);
    } catch (const c10::OutOfMemoryError &) {
        return {};
    }
}

// dybit_gemm: on the current stream a product that uses a workspace gets it (dybit_gemm_work).
template <size_t... I>
std::tuple<std::tuple_element_t<I, Entry<&dybit_gemm>::Arguments>...> front(const Entry<&dybit_gemm>::Arguments &a, std::index_sequence<I...>)
{
    return {std::get<I>(a)...};
}
PyObject *gemm(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    using Gemm = Entry<&dybit_gemm>;
    constexpr size_t kStream = Gemm::kCount - 1;
    HANDLE_TH_ERRORS
    if (n != Gemm::kCount || args[kStream] != Py_None) return Gemm::call(self, args, n);
    try {
        const Gemm::Arguments a = Gemm::arguments(args);
        const bool results = std::get<11>(a) != nullptr;                 // else the call is refused
        const size_t need = results ? dybit_gemm_workspace_bytes(std::get<0>(a), std::get<1>(a), std::get<2>(a), std::get<4>(a), std::get<7>(a)) : 0;
        const c10::DataPtr work = need ? scratch(need) : c10::DataPtr();
        if (!work) return PyLong_FromLong((long)Gemm::run(a));
        const auto with_work = std::tuple_cat(front(a, std::make_index_sequence<kStream>{}),
                                              std::tuple<uint8_t *, size_t, dybit_stream>{(uint8_t *)work.get(), need, std::get<kStream>(a)});
        return PyLong_FromLong((long)Entry<&dybit_gemm_work>::run(with_work));
    } catch (const PythonError &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// empty(like, floats, *sizes): an uninitialised tensor of float32 (or, floats false, bytes) on the device of `like`.
PyObject *empty(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n < 3) { PyErr_SetString(PyExc_TypeError, "empty(like, floats, *sizes)"); return nullptr; }
    try {
        if (!THPVariable_Check(args[0])) { PyErr_SetString(PyExc_TypeError, "expected a tensor"); return nullptr; }
        c10::SmallVector<int64_t, 4> sizes;
        for (Py_ssize_t i = 2; i < n; ++i) sizes.push_back(integer(args[i]));
        const auto options = at::TensorOptions().device(THPVariable_Unpack(args[0]).device()).dtype(truth(args[1]) ? at::kFloat : at::kByte);
        return THPVariable_Wrap(at::empty(sizes, options));
    } catch (const PythonError &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// dybit_packed_bytes((bits, signed), n)
PyObject *packed_bytes(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 2) { PyErr_SetString(PyExc_TypeError, "expected 2 arguments"); return nullptr; }
    try {
        const dybit_fmt f = format(args[0]);
        return PyLong_FromSize_t(dybit_packed_bytes(f, (size_t)integer(args[1])));
    } catch (const PythonError &) {
        return nullptr;
    }
}

#define DYBIT_ENTRY(name) {#name, (PyCFunction)(void (*)(void))Entry<&name>::call, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    DYBIT_ENTRY(dybit_absmax_scale), DYBIT_ENTRY(dybit_absmax_scale_ws), DYBIT_ENTRY(dybit_scale_from_absmax),
    DYBIT_ENTRY(dybit_quantize), DYBIT_ENTRY(dybit_quantize_absmax), DYBIT_ENTRY(dybit_quantize_pad),
    DYBIT_ENTRY(dybit_quantize_rows), DYBIT_ENTRY(dybit_quantize_cols), DYBIT_ENTRY(dybit_dequantize),
    DYBIT_ENTRY(dybit_fake_quant), DYBIT_ENTRY(dybit_fake_quant_bwd), DYBIT_ENTRY(dybit_rmse),
    {"dybit_gemm", (PyCFunction)(void (*)(void))gemm, METH_FASTCALL, nullptr}, DYBIT_ENTRY(dybit_gemm_ex), DYBIT_ENTRY(dybit_gemm_wb), DYBIT_ENTRY(dybit_gemm_wb_rc), DYBIT_ENTRY(dybit_gemm_pc),
    DYBIT_ENTRY(dybit_conv2d), DYBIT_ENTRY(dybit_conv2d_ex), DYBIT_ENTRY(dybit_conv2d_wb), DYBIT_ENTRY(dybit_conv2d_wb_rc), DYBIT_ENTRY(dybit_conv2d_pc),
    DYBIT_ENTRY(dybit_dwconv2d), DYBIT_ENTRY(dybit_dwconv2d_wb), DYBIT_ENTRY(dybit_group_conv2d), DYBIT_ENTRY(dybit_maxpool2d_codes),
    {"dybit_packed_bytes", (PyCFunction)(void (*)(void))packed_bytes, METH_FASTCALL, nullptr},
    {"empty", (PyCFunction)(void (*)(void))empty, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
