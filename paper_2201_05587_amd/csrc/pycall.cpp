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

// What the binding hands over once.
PyObject *conv_shape_type, *gemm_shape_type, *schedule_type;
PyObject *refuse_struct;  // (object, expected type): raises what ctypes raises for such an argument

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

const at::Tensor *tensor_or_null(PyObject *o, const char *name)
{
    if (o == Py_None) return nullptr;
    TORCH_CHECK_TYPE(THPVariable_Check(o), name, " must be a tensor");
    return &THPVariable_Unpack(o);
}

void *data_of(const at::Tensor *t) { return t ? t->data_ptr() : nullptr; }

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

// Plan, workspace, launch.  Returns the output tensor, or the status as a Python integer.
PyObject *call(int cls, const void *shape, PyObject *sched, OpPointers p, PyObject *ws, const at::Tensor &out, PyObject *y)
{
    int rc = TT_OK;
    at::Tensor own_ws;
    PreparedOp op;
    {
        tt_schedule rec;
        if (sched != Py_None) rec = struct_of<tt_schedule>(sched, schedule_type);
        const at::Tensor *given = tensor_or_null(ws, "ws");
        if (given) {
            p.ws = given->data_ptr();
            p.ws_bytes = given->nbytes();
        }
        rc = check_op_pointers(cls, p);
        if (rc == TT_OK) rc = prepare_op(sched != Py_None ? &rec : nullptr, cls, shape, &op);
        if (rc == TT_OK && !given && op.plan.workspace_bytes > 0) {
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
    if (rc != TT_OK) return PyLong_FromLong(rc);
    if (y != Py_None) {
        Py_INCREF(y);
        return y;
    }
    return THPVariable_Wrap(out);
}

// conv2d(x, w, bias, residual, shape, cls, sched, ws, y)
PyObject *py_conv2d(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    TORCH_CHECK_TYPE(n == 9, "conv2d takes nine arguments");
    const at::Tensor *x = tensor_or_null(a[0], "x"), *w = tensor_or_null(a[1], "w"), *b = tensor_or_null(a[2], "bias"),
                     *r = tensor_or_null(a[3], "residual"), *y = tensor_or_null(a[8], "y");
    const tt_conv_shape s = struct_of<tt_conv_shape>(a[4], conv_shape_type);
    const long cls = PyLong_AsLong(a[5]);
    if (cls == -1 && PyErr_Occurred()) throw python_error();
    TORCH_CHECK_TYPE(x, "x must be a tensor");
    at::Tensor out;
    const int64_t ho = out_extent(s.h, s.pad_h, s.r, s.stride_h), wo = out_extent(s.w, s.pad_w, s.s, s.stride_w);
    if (!y) out = at::empty({s.n, s.k, ho, wo}, x->options());
    if (!is_conv_class((int)cls)) return PyLong_FromLong(TT_ERR_BAD_ARG);
    return call((int)cls, &s, a[6], {x->data_ptr(), data_of(w), data_of(b), data_of(r), y ? y->data_ptr() : out.data_ptr(), nullptr, 0},
                a[7], out, a[8]);
    END_HANDLE_TH_ERRORS
}

// dense(x, w, bias, shape, cls, sched, ws, y)
PyObject *py_dense(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    TORCH_CHECK_TYPE(n == 8, "dense takes eight arguments");
    const at::Tensor *x = tensor_or_null(a[0], "x"), *w = tensor_or_null(a[1], "w"), *b = tensor_or_null(a[2], "bias"),
                     *y = tensor_or_null(a[7], "y");
    const tt_gemm_shape s = struct_of<tt_gemm_shape>(a[3], gemm_shape_type);
    const long cls = PyLong_AsLong(a[4]);
    if (cls == -1 && PyErr_Occurred()) throw python_error();
    TORCH_CHECK_TYPE(x, "x must be a tensor");
    at::Tensor out;
    if (!y) out = at::empty({s.m, s.n}, x->options());
    if (!is_dense_class((int)cls)) return PyLong_FromLong(TT_ERR_BAD_ARG);
    return call((int)cls, &s, a[5], {x->data_ptr(), data_of(w), data_of(b), nullptr, y ? y->data_ptr() : out.data_ptr(), nullptr, 0}, a[6],
                out, a[7]);
    END_HANDLE_TH_ERRORS
}

// matmul(a, b, shape, sched, ws, c)
PyObject *py_matmul(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    TORCH_CHECK_TYPE(n == 6, "matmul takes six arguments");
    const at::Tensor *x = tensor_or_null(a[0], "a"), *w = tensor_or_null(a[1], "b"), *y = tensor_or_null(a[5], "c");
    const tt_gemm_shape s = struct_of<tt_gemm_shape>(a[2], gemm_shape_type);
    TORCH_CHECK_TYPE(x, "a must be a tensor");
    at::Tensor out;
    if (!y) out = at::empty({s.batch, s.m, s.n}, x->options());
    return call(TT_BATCH_MATMUL, &s, a[3], {x->data_ptr(), data_of(w), nullptr, nullptr, y ? y->data_ptr() : out.data_ptr(), nullptr, 0},
                a[4], out, a[5]);
    END_HANDLE_TH_ERRORS
}

// dwconv(x, w, bias, shape, sched, y)
PyObject *py_dwconv(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    TORCH_CHECK_TYPE(n == 6, "dwconv takes six arguments");
    const at::Tensor *x = tensor_or_null(a[0], "x"), *w = tensor_or_null(a[1], "w"), *b = tensor_or_null(a[2], "bias"),
                     *y = tensor_or_null(a[5], "y");
    const tt_conv_shape s = struct_of<tt_conv_shape>(a[3], conv_shape_type);
    TORCH_CHECK_TYPE(x, "x must be a tensor");
    at::Tensor out;
    const int64_t ho = out_extent(s.h, s.pad_h, s.r, s.stride_h), wo = out_extent(s.w, s.pad_w, s.s, s.stride_w);
    if (!y) out = at::empty({s.n, s.c, ho, wo}, x->options());
    return call(TT_DWCONV_BIAS_RELU6, &s, a[4],
                {x->data_ptr(), data_of(w), data_of(b), nullptr, y ? y->data_ptr() : out.data_ptr(), nullptr, 0}, Py_None, out, a[5]);
    END_HANDLE_TH_ERRORS
}

// bind(conv shape type, gemm shape type, schedule type, refuse_struct): once, by the binding
PyObject *py_bind(PyObject *, PyObject *args)
{
    PyObject *o[4];
    if (!PyArg_ParseTuple(args, "OOOO", &o[0], &o[1], &o[2], &o[3])) return nullptr;
    PyObject **const slots[4] = {&conv_shape_type, &gemm_shape_type, &schedule_type, &refuse_struct};
    for (int i = 0; i < 4; ++i) {
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
