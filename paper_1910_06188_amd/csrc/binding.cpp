// Python entry points of the C ABI (include/q8.h): tensors to device pointers, numbers to the types of the declaration, the
// call with the interpreter lock released.  Nothing else happens here; sizes are checked by the Python functions in front.
//
// A call of a small layer is bound by the host: a kernel launch takes 3.5 us of it, and reading twelve tensors through three
// attribute calls each and handing eighteen arguments to ctypes took another 2.0 to 2.4.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "q8.h"

namespace {

// One argument.  On failure a Python error is set.
template <class T>
T argument(PyObject* o)
{
    if constexpr (std::is_pointer_v<T>) {
        if (o == Py_None) return nullptr;
        if (!THPVariable_Check(o)) {
            PyErr_SetString(PyExc_TypeError, "q8 takes tensors");
            return nullptr;
        }
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda())
            PyErr_SetString(PyExc_ValueError, "q8 takes device tensors");
        else if (!t.is_contiguous())
            PyErr_SetString(PyExc_ValueError, "q8 takes contiguous tensors");
        else
            return static_cast<T>(t.data_ptr());
        return nullptr;
    } else if constexpr (std::is_floating_point_v<T>) {
        return static_cast<T>(PyFloat_AsDouble(o));
    } else {
        return static_cast<T>(PyLong_AsUnsignedLongLongMask(o));
    }
}

// The stream, the last parameter of every function, comes as its raw handle; None is torch's current one.
void* stream_of(PyObject* o)
{
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    return reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(o)));
}

template <auto kFunction, class... A, size_t... I>
PyObject* call(PyObject* const* args, q8_status (*)(A...), std::index_sequence<I...>)
{
    using Params = std::tuple<A...>;
    Params p;
    constexpr size_t kStream = sizeof...(A) - 1;
    const auto convert = [&](auto index) {
        constexpr size_t i = decltype(index)::value;
        if constexpr (i == kStream)
            std::get<i>(p) = stream_of(args[i]);
        else
            std::get<i>(p) = argument<std::tuple_element_t<i, Params>>(args[i]);
        return PyErr_Occurred() == nullptr;
    };
    if (!(convert(std::integral_constant<size_t, I>{}) && ...)) return nullptr;
    q8_status status;
    Py_BEGIN_ALLOW_THREADS
    status = std::apply(kFunction, p);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(static_cast<long>(status));
}

template <class... A>
constexpr size_t arity(q8_status (*)(A...))
{
    return sizeof...(A);
}

template <auto kFunction>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    constexpr size_t kArgs = arity(kFunction);
    if (n != static_cast<Py_ssize_t>(kArgs)) return PyErr_Format(PyExc_TypeError, "takes %zu arguments, got %zd", kArgs, n);
    try {
        return call<kFunction>(args, kFunction, std::make_index_sequence<kArgs>{});
    } catch (const std::exception& e) {  // a tensor without storage of its own (under a functional transform)
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

#define Q8_ENTRY(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<&NAME>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {Q8_ENTRY(q8_absmax),
                         Q8_ENTRY(q8_scale_from_amax),
                         Q8_ENTRY(q8_quantize),
                         Q8_ENTRY(q8_quantize_amax),
                         Q8_ENTRY(q8_quantize_dynamic),
                         Q8_ENTRY(q8_linear),
                         Q8_ENTRY(q8_linear_residual),
                         Q8_ENTRY(q8_linear_f32),
                         Q8_ENTRY(q8_linear_f32_static),
                         Q8_ENTRY(q8_linear_f32_slots),
                         Q8_ENTRY(q8_embedding),
                         Q8_ENTRY(q8_embedding_sum3),
                         Q8_ENTRY(q8_fake_quantize),
                         Q8_ENTRY(q8_ema_update),
                         Q8_ENTRY(q8_fake_quantize_ema),
                         Q8_ENTRY(q8_ste_backward),
                         Q8_ENTRY(q8_layernorm_absmax),
                         Q8_ENTRY(q8_embedding_sum3_layernorm),
                         Q8_ENTRY(q8_attention),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
