// The calls a model makes for every layer - quantize, linear, both in one - from Python objects to the C ABI without
// ctypes: checks, allocations and pointers in native code.  Small calls are bound by the host: through ctypes
// linear_fp16 of one token took 9.6 us, linear (two calls) 16.1, of which the launches are 3.2 each; here 5.7 and 10.2.  77
// tokens through a layer of K = 1920, N = 3003 by two calls 16.4 -> 10.9 us, a token through the 8B block 36.5 -> 34.3, where
// its kernels (31.5 us) are the bound.  The library's functions come in as addresses, so that whichever build of it the
// package has loaded is the one that runs.  Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "mixllm.h"

namespace {

namespace py = pybind11;

decltype(&mixllm_query_sizes) query_sizes;
decltype(&mixllm_quantize_activations) quantize_activations;
decltype(&mixllm_mixed_linear_path) mixed_linear_path;
decltype(&mixllm_mixed_linear_fp16) mixed_linear_fp16;

struct Refused {   // what an assertion of the Python side would say
    const char *what;
};

// the tensor behind an argument, or an undefined one for None
at::Tensor tensor(PyObject *o)
{
    if (o == Py_None) return at::Tensor();
    TORCH_CHECK_TYPE(THPVariable_Check(o), "expected a tensor, got ", Py_TYPE(o)->tp_name);
    return THPVariable_Unpack(o);
}

// device address of a tensor's data; null for none and for an empty one
void *address(const at::Tensor &t)
{
    if (!t.defined() || t.numel() == 0) return nullptr;
    if (!t.is_cuda() || !t.is_contiguous()) throw Refused{"device, contiguous tensors only"};
    return t.data_ptr();
}

int32_t index(PyObject *o)
{
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw python_error();
    return (int32_t)v;
}

// a descriptor's field: whatever int() makes a number of
int32_t number(PyObject *o)
{
    if (PyLong_CheckExact(o)) return index(o);
    const py::object i = py::reinterpret_steal<py::object>(PyNumber_Long(o));
    if (!i) throw python_error();
    return index(i.ptr());
}

// K, N, n8, w8_group, w8, w4, s8, s4, z4, perm of a packed layer, as they stand in the arguments
struct Layer {
    int32_t K, N, n8, w8_group;
    at::Tensor w8, w4, s8, s4, z4, perm;
    explicit Layer(PyObject *const *a)
        : K(number(a[0])), N(number(a[1])), n8(number(a[2])), w8_group(number(a[3])), w8(tensor(a[4])), w4(tensor(a[5])), s8(tensor(a[6])),
          s4(tensor(a[7])), z4(tensor(a[8])), perm(tensor(a[9]))
    {
    }
};

void half_matrix(const at::Tensor &x)
{
    if (!x.defined() || x.scalar_type() != at::kHalf || x.dim() != 2) throw Refused{"x: an fp16 matrix"};
}

// A buffer of the caller's holds `n` values of `type`, or the same number of integers of that width (raw bits): what the
// kernels read and write goes by the sizes of the call alone.  A missing buffer is left to the library.
void holds(const at::Tensor &t, at::ScalarType type, int64_t n, const char *what)
{
    if (!t.defined()) return;
    const bool bits = at::isIntegralType(t.scalar_type(), /*includeBool=*/true) && t.itemsize() == (int64_t)at::elementSize(type);
    if ((t.scalar_type() != type && !bits) || t.numel() < n) throw Refused{what};
}

// A subclass of Tensor, or a mode, may have a new_empty of its own: results are then allocated by it, so that they are of
// the type they would have in Python.
bool overrides_new_empty(PyObject *o)
{
    return !THPVariable_CheckExact(o) || at::impl::torch_function_mode_enabled();
}
at::Tensor new_empty_in_python(PyObject *o, int64_t rows, int64_t columns, at::ScalarType type)
{
    const auto dtype = py::reinterpret_borrow<py::object>((PyObject *)torch::getTHPDtype(type));
    return tensor(py::handle(o).attr("new_empty")(py::make_tuple(rows, columns), py::arg("dtype") = dtype).ptr());
}

// f() with its C++ exceptions as Python ones.  The calls below release the interpreter while they allocate and launch; a
// status other than MIXLLM_OK comes back as a number.
template <typename F>
PyObject *run(Py_ssize_t n, Py_ssize_t expected, F &&f)
{
    HANDLE_TH_ERRORS
    TORCH_CHECK_TYPE(n == expected, "expected ", expected, " arguments, got ", n);
    try {
        return f();
    } catch (const Refused &r) {
        PyErr_SetString(PyExc_AssertionError, r.what);
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// (A workspace's element count stands for its bytes: exact for the uint8 tensor it is meant to be, short of them, never
// beyond, for any other.)

// linear_fp16(x, <layer>, act_group, out, workspace, stream) -> y, or a status
PyObject *py_linear_fp16(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return run(n, 15, [&]() -> PyObject * {
        const at::Tensor x = tensor(a[0]);
        const Layer L(a + 1);
        const int32_t act_group = number(a[11]);
        at::Tensor y = tensor(a[12]), ws = tensor(a[13]);
        void *stream = PyLong_AsVoidPtr(a[14]);
        half_matrix(x);
        holds(y, at::kHalf, x.size(0) * L.N, "y: an fp16 buffer of tokens x outputs");
        if (x.size(1) != L.K) throw Refused{"x has as many columns as the layer has inputs"};
        if (!y.defined() && overrides_new_empty(a[0])) y = new_empty_in_python(a[0], x.size(0), L.N, at::kHalf);
        int rc;
        {
            py::gil_scoped_release no_gil;
            const mixllm_desc d{(int32_t)x.size(0), L.K, L.N, L.n8, MIXLLM_GROUP, act_group, L.w8_group};
            if (!y.defined()) y = x.new_empty({x.size(0), L.N});
            rc = MIXLLM_OK;
            if (!ws.defined()) {
                mixllm_sizes s;
                rc = query_sizes(&d, &s);
                if (rc == MIXLLM_OK) ws = x.new_empty({(int64_t)s.workspace_bytes}, x.options().dtype(at::kByte));
            }
            if (rc == MIXLLM_OK)
                rc = mixed_linear_fp16(&d, address(x), address(L.w4), address(L.w8), address(L.s4), address(L.s8), address(L.z4),
                                       (const int32_t *)address(L.perm), address(y), address(ws), (size_t)ws.numel(), stream);
        }
        return rc == MIXLLM_OK ? THPVariable_Wrap(std::move(y)) : PyLong_FromLong(rc);
    });
}

// quantize_activations(x, act_group or None, (xq, xs) or None, stream) -> (xq, xs), or a status.  Only where no buffers are
// given at all are they allocated: one that is missing from a pair is refused by the library.
PyObject *py_quantize_activations(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return run(n, 4, [&]() -> PyObject * {
        const at::Tensor x = tensor(a[0]);
        const bool per_token = a[1] == Py_None, allocate = a[2] == Py_None;
        int32_t act_group = per_token ? 0 : allocate ? index(a[1]) : number(a[1]);   // (a tensor's size is an integer)
        at::Tensor xq, xs;
        if (!allocate) {
            const py::object out = py::reinterpret_steal<py::object>(PySequence_Tuple(a[2]));
            if (!out) throw python_error();
            TORCH_CHECK_VALUE(PyTuple_GET_SIZE(out.ptr()) == 2, "out: two buffers, got ", PyTuple_GET_SIZE(out.ptr()));
            xq = tensor(PyTuple_GET_ITEM(out.ptr(), 0));
            xs = tensor(PyTuple_GET_ITEM(out.ptr(), 1));
        }
        void *stream = PyLong_AsVoidPtr(a[3]);
        half_matrix(x);
        const int32_t M = (int32_t)x.size(0), K = (int32_t)x.size(1);
        if (per_token) act_group = K;
        holds(xq, at::kChar, (int64_t)M * K, "xq: an int8 buffer of tokens x inputs");
        if (act_group > 0) holds(xs, at::kHalf, (int64_t)M * (K / act_group), "xs: an fp16 buffer of tokens x groups");
        if (allocate && act_group <= 0) throw Refused{"act_group is positive"};
        if (allocate && overrides_new_empty(a[0])) {
            xq = new_empty_in_python(a[0], M, K, at::kChar);
            xs = new_empty_in_python(a[0], M, K / act_group, at::kHalf);
        }
        int rc;
        {
            py::gil_scoped_release no_gil;
            if (allocate && !xq.defined()) {
                xq = x.new_empty({M, K}, x.options().dtype(at::kChar));
                xs = x.new_empty({M, K / act_group});
            }
            const mixllm_desc d{M, K, 1, 0, MIXLLM_GROUP, act_group, K};
            rc = quantize_activations(&d, address(x), (int8_t *)address(xq), address(xs), stream);
        }
        if (rc != MIXLLM_OK) return PyLong_FromLong(rc);
        PyObject *q = THPVariable_Wrap(std::move(xq));
        PyObject *s = q ? THPVariable_Wrap(std::move(xs)) : nullptr;
        PyObject *both = s ? PyTuple_Pack(2, q, s) : nullptr;
        Py_XDECREF(q);
        Py_XDECREF(s);
        return both;
    });
}

// mixed_linear(xq, xs, <layer>, path, out, workspace, stream) -> y, or a status
PyObject *py_mixed_linear(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return run(n, 16, [&]() -> PyObject * {
        const at::Tensor xq = tensor(a[0]), xs = tensor(a[1]);
        const Layer L(a + 2);
        const int32_t path = index(a[12]);
        at::Tensor y = tensor(a[13]);
        const at::Tensor ws = tensor(a[14]);
        void *stream = PyLong_AsVoidPtr(a[15]);
        if (!xq.defined() || xq.dim() != 2) throw Refused{"xq: a matrix"};
        const int64_t M = xq.size(0), K = xq.size(1);
        if (K != L.K || xs.size(0) != M) throw Refused{"xq, xs and the layer agree in their sizes"};
        if (xs.size(1) == 0) throw Refused{"xs has a column"};
        const int32_t act_group = (int32_t)(K / xs.size(1));
        holds(xq, at::kChar, M * K, "xq: an int8 matrix");
        if (act_group == K || act_group == MIXLLM_GROUP) {
            // as many scales as the library reads: 129 columns for 130 groups also divide to groups of 128
            holds(xs, at::kHalf, M * (K / act_group), "xs: fp16 scales, tokens x groups");
            if (xs.numel() != M * (K / act_group)) throw Refused{"xs: one scale per token and group"};
        }
        holds(y, at::kHalf, M * L.N, "y: an fp16 buffer of tokens x outputs");
        if (!y.defined() && overrides_new_empty(a[0])) y = new_empty_in_python(a[0], M, L.N, at::kHalf);
        int rc;
        {
            py::gil_scoped_release no_gil;
            if (!y.defined()) y = xq.new_empty({M, L.N}, xq.options().dtype(at::kHalf));
            const mixllm_desc d{(int32_t)M, L.K, L.N, L.n8, MIXLLM_GROUP, act_group, L.w8_group};
            rc = mixed_linear_path(&d, (const int8_t *)address(xq), address(xs), address(L.w4), address(L.w8), address(L.s4), address(L.s8),
                                   address(L.z4), (const int32_t *)address(L.perm), address(y), address(ws),
                                   ws.defined() ? (size_t)ws.numel() : 0, path, stream);
        }
        return rc == MIXLLM_OK ? THPVariable_Wrap(std::move(y)) : PyLong_FromLong(rc);
    });
}

// bind(query_sizes, quantize_activations, mixed_linear_path, mixed_linear_fp16): addresses of the library's functions
PyObject *py_bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return run(n, 4, [&]() -> PyObject * {
        query_sizes = (decltype(query_sizes))PyLong_AsVoidPtr(a[0]);
        quantize_activations = (decltype(quantize_activations))PyLong_AsVoidPtr(a[1]);
        mixed_linear_path = (decltype(mixed_linear_path))PyLong_AsVoidPtr(a[2]);
        mixed_linear_fp16 = (decltype(mixed_linear_fp16))PyLong_AsVoidPtr(a[3]);
        Py_RETURN_NONE;
    });
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)())py_bind, METH_FASTCALL, nullptr},
    {"linear_fp16", (PyCFunction)(void (*)())py_linear_fp16, METH_FASTCALL, nullptr},
    {"quantize_activations", (PyCFunction)(void (*)())py_quantize_activations, METH_FASTCALL, nullptr},
    {"mixed_linear", (PyCFunction)(void (*)())py_mixed_linear, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) { return PyModule_Create(&module); }
