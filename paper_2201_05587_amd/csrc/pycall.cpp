// Operator calls from Python without an interpreter in between: reads the tensors, the shape and the record,
// lays out the plan, allocates the output and the split-K workspace where the caller gave none, and launches.
//
// A small kernel runs for 4 to 6 us.  Marshalled in Python (a plan for the workspace size, eleven ctypes
// arguments, the stream lookup, a second plan inside the entry point) its call took 10 to 12 us of host time, so
// a program's small calls ran at the interpreter's pace; from here a call takes about 3 us, most of it the
// runtime's launch.
//
// The functions mirror the wrappers of api.py, which pass their arguments on and raise TTError for a status.
#include <Python.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "tt_internal.h"

using namespace tt;

namespace {

// What the binding hands over once: its structure types, and functions for what is rare enough for Python.
PyObject *conv_shape_type, *gemm_shape_type, *schedule_type;
PyObject *refuse_struct;  // (object, expected type): raises what ctypes raises for such an argument
PyObject *empty_tensor;   // (x, sizes): an output of x's type and place

// A reference that ends with the scope.
class Owned {
public:
    explicit Owned(PyObject *o) : o_(o)
    {
        if (!o) throw python_error();
    }
    ~Owned() { Py_DECREF(o_); }
    Owned(const Owned &) = delete;
    Owned &operator=(const Owned &) = delete;
    PyObject *get() const { return o_; }

private:
    PyObject *o_;
};

// The contents of a ctypes structure of one type (or a type derived from it): a buffer of the right size alone could be a
// structure of another layout.
template <class T> T struct_of(PyObject *obj, PyObject *type)
{
    TORCH_CHECK(type, "_ttcall is used through the binding");
    int ok = (PyObject *)Py_TYPE(obj) == type;
    if (!ok) ok = PyObject_IsInstance(obj, type);
    if (ok < 0) throw python_error();
    if (!ok) {
        Owned unreachable(PyObject_CallFunctionObjArgs(refuse_struct, obj, type, nullptr));
        TORCH_CHECK_TYPE(false, "wrong type");
    }
    Py_buffer view;
    if (PyObject_GetBuffer(obj, &view, PyBUF_SIMPLE) != 0) throw python_error();
    const bool whole = (size_t)view.len >= sizeof(T);
    T out{};
    if (whole) out = *static_cast<const T *>(view.buf);
    PyBuffer_Release(&view);
    TORCH_CHECK_TYPE(whole, "structure without its contents");
    return out;
}

// Address of an argument: null for None, and for anything but a plain tensor what its own data_ptr() says.
void *address_of(PyObject *o)
{
    if (o == Py_None) return nullptr;
    if (THPVariable_CheckExact(o)) return THPVariable_Unpack(o).data_ptr();
    Owned at(PyObject_CallMethod(o, "data_ptr", nullptr));
    if (at.get() == Py_None) return nullptr;
    void *const p = PyLong_AsVoidPtr(at.get());
    if (!p && PyErr_Occurred()) throw python_error();
    return p;
}

int64_t integer_from(PyObject *o, const char *method)
{
    Owned v(PyObject_CallMethod(o, method, nullptr));
    const long long n = PyLong_AsLongLong(v.get());
    if (n == -1 && PyErr_Occurred()) throw python_error();
    return n;
}
size_t bytes_of(PyObject *o)
{
    if (THPVariable_CheckExact(o)) return THPVariable_Unpack(o).nbytes();
    return (size_t)(integer_from(o, "numel") * integer_from(o, "element_size"));
}

// The output of a call: the caller's, or a new one of x's type and place, which becomes a Python object behind the launch.
class Output {
public:
    Output(PyObject *given, PyObject *x, at::IntArrayRef sizes)
    {
        if (given != Py_None) {
            object_ = Py_NewRef(given);
        } else if (THPVariable_CheckExact(x)) {
            made_ = at::empty(sizes, THPVariable_Unpack(x).options());
        } else {
            Owned tuple(PyTuple_New((Py_ssize_t)sizes.size()));
            for (size_t i = 0; i < sizes.size(); ++i) PyTuple_SET_ITEM(tuple.get(), i, PyLong_FromLongLong(sizes[i]));
            object_ = PyObject_CallFunctionObjArgs(empty_tensor, x, tuple.get(), nullptr);
            if (!object_) throw python_error();
        }
    }
    ~Output() { Py_XDECREF(object_); }
    Output(const Output &) = delete;
    Output &operator=(const Output &) = delete;
    void *address() const { return object_ ? address_of(object_) : made_.data_ptr(); }
    PyObject *result() { return object_ ? Py_NewRef(object_) : THPVariable_Wrap(std::move(made_)); }

private:
    PyObject *object_ = nullptr;
    at::Tensor made_;
};

int class_of(PyObject *o)
{
    const long cls = PyLong_AsLong(o);
    if (cls == -1 && PyErr_Occurred()) throw python_error();
    return (int)cls;
}

int64_t out_extent(int64_t in, int64_t pad, int64_t filter, int64_t stride)
{
    const int64_t n = in + 2 * pad - filter;
    if (stride == 0) {
        PyErr_SetString(PyExc_ZeroDivisionError, "integer division or modulo by zero");
        throw python_error();
    }
    return n / stride - (n % stride != 0 && (n < 0) != (stride < 0)) + 1; // rounded down
}

void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Plan, workspace, launch.  Returns the output, or the status as a Python integer.
PyObject *call(int cls, const void *shape, PyObject *sched, OpPointers p, PyObject *ws, Output &out)
{
    int rc = TT_OK;
    at::Tensor own_ws;
    PreparedOp op;
    {
        tt_schedule rec;
        if (sched != Py_None) rec = struct_of<tt_schedule>(sched, schedule_type);
        if (ws != Py_None) {
            p.ws = address_of(ws);
            p.ws_bytes = bytes_of(ws);
        }
        p.out = out.address();
        rc = check_op_pointers(cls, p);
        if (rc == TT_OK) rc = prepare_op(sched != Py_None ? &rec : nullptr, cls, shape, &op);
        if (rc == TT_OK && ws == Py_None && op.plan.workspace_bytes > 0) {
            own_ws = at::empty({op.plan.workspace_bytes}, at::TensorOptions().dtype(at::kByte).device(at::kCUDA));
            p.ws = own_ws.data_ptr();
            p.ws_bytes = (size_t)op.plan.workspace_bytes;
        }
    }
    if (rc == TT_OK) {
        void *const stream = current_stream();
        Py_BEGIN_ALLOW_THREADS rc = launch_op(op, &p, 1, stream); // (a full queue makes a launch wait)
        Py_END_ALLOW_THREADS
    }
    return rc == TT_OK ? out.result() : PyLong_FromLong(rc);
}

// conv2d(x, w, bias, residual, shape, cls, sched, ws, y)
PyObject *py_conv2d(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    TORCH_CHECK_TYPE(n == 9, "conv2d takes nine arguments");
    const tt_conv_shape s = struct_of<tt_conv_shape>(a[4], conv_shape_type);
    const int cls = class_of(a[5]);
    const int64_t ho = out_extent(s.h, s.pad_h, s.r, s.stride_h), wo = out_extent(s.w, s.pad_w, s.s, s.stride_w);
    Output out(a[8], a[0], {s.n, s.k, ho, wo});
    if (!is_conv_class(cls)) return PyLong_FromLong(TT_ERR_BAD_ARG);
    return call(cls, &s, a[6], {address_of(a[0]), address_of(a[1]), address_of(a[2]), address_of(a[3]), nullptr, nullptr, 0}, a[7], out);
    END_HANDLE_TH_ERRORS
}

// dense(x, w, bias, shape, cls, sched, ws, y)
PyObject *py_dense(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    TORCH_CHECK_TYPE(n == 8, "dense takes eight arguments");
    const tt_gemm_shape s = struct_of<tt_gemm_shape>(a[3], gemm_shape_type);
    const int cls = class_of(a[4]);
    Output out(a[7], a[0], {s.m, s.n});
    if (!is_dense_class(cls)) return PyLong_FromLong(TT_ERR_BAD_ARG);
    return call(cls, &s, a[5], {address_of(a[0]), address_of(a[1]), address_of(a[2]), nullptr, nullptr, nullptr, 0}, a[6], out);
    END_HANDLE_TH_ERRORS
}

// matmul(a, b, shape, sched, ws, c)
PyObject *py_matmul(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    TORCH_CHECK_TYPE(n == 6, "matmul takes six arguments");
    const tt_gemm_shape s = struct_of<tt_gemm_shape>(a[2], gemm_shape_type);
    Output out(a[5], a[0], {s.batch, s.m, s.n});
    return call(TT_BATCH_MATMUL, &s, a[3], {address_of(a[0]), address_of(a[1]), nullptr, nullptr, nullptr, nullptr, 0}, a[4], out);
    END_HANDLE_TH_ERRORS
}

// dwconv(x, w, bias, shape, sched, y)
PyObject *py_dwconv(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    TORCH_CHECK_TYPE(n == 6, "dwconv takes six arguments");
    const tt_conv_shape s = struct_of<tt_conv_shape>(a[3], conv_shape_type);
    const int64_t ho = out_extent(s.h, s.pad_h, s.r, s.stride_h), wo = out_extent(s.w, s.pad_w, s.s, s.stride_w);
    Output out(a[5], a[0], {s.n, s.c, ho, wo});
    return call(TT_DWCONV_BIAS_RELU6, &s, a[4], {address_of(a[0]), address_of(a[1]), address_of(a[2]), nullptr, nullptr, nullptr, 0}, Py_None, out);
    END_HANDLE_TH_ERRORS
}

// bind(conv shape type, gemm shape type, schedule type, refuse_struct, empty_tensor): once, by the binding
PyObject *py_bind(PyObject *, PyObject *args)
{
    PyObject *o[5];
    if (!PyArg_ParseTuple(args, "OOOOO", &o[0], &o[1], &o[2], &o[3], &o[4])) return nullptr;
    PyObject **const slots[5] = {&conv_shape_type, &gemm_shape_type, &schedule_type, &refuse_struct, &empty_tensor};
    for (int i = 0; i < 5; ++i) {
        PyObject *const before = *slots[i];
        *slots[i] = Py_NewRef(o[i]);
        Py_XDECREF(before);
    }
    Py_RETURN_NONE;
}

// The handle of the current stream of the current device.
PyObject *py_stream(PyObject *, PyObject *)
{
    HANDLE_TH_ERRORS
    return PyLong_FromVoidPtr(current_stream());
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"bind", py_bind, METH_VARARGS, nullptr},
    {"conv2d", (PyCFunction)(void (*)())py_conv2d, METH_FASTCALL, nullptr},
    {"dense", (PyCFunction)(void (*)())py_dense, METH_FASTCALL, nullptr},
    {"matmul", (PyCFunction)(void (*)())py_matmul, METH_FASTCALL, nullptr},
    {"dwconv", (PyCFunction)(void (*)())py_dwconv, METH_FASTCALL, nullptr},
    {"stream", py_stream, METH_NOARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ttcall", "Operator calls of libtt.", -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__ttcall(void) { return PyModule_Create(&module); }
