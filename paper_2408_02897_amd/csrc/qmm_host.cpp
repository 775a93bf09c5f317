// The binding's short path: quantized_operand / scale_quantize, gemm and metric of qmm.py for plain tensors, as one native call
// each -- descriptors, outputs and workspace from torch's allocator, the size query and the call on the current stream.  What a
// small product takes is the host's time: as ctypes calls the four calls of one linear layer took 27 us around 12 us of
// launches.  Every function returns None where its arguments are not the plain case (tensor subclasses, another device or
// type, shapes that do not fit, flags it does not know, an active torch function mode): qmm.py then goes its own way, which
// also raises the errors.  A failed status comes back as a number.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "qmm.h"

namespace {

PyTypeObject* operand_type = nullptr;          // qmm.Operand, the ctypes structure of a qmm_operand

// Without the interpreter's lock, as ctypes calls run.
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

bool plain(PyObject* o) { return THPVariable_CheckExact(o); }
bool modes_active() { return at::impl::PythonTorchFunctionTLS::stack_len() > 0; }
bool number(PyObject* o, int64_t* v)
{
    if (!PyLong_Check(o)) return false;        // (bool among them)
    int overflow = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
bool dtype_of(const at::Tensor& x, int32_t* d)
{
    if (x.scalar_type() == at::kBFloat16) *d = QMM_DT_BF16;
    else if (x.scalar_type() == at::kFloat) *d = QMM_DT_F32;
    else return false;
    return true;
}
bool describe(const at::Tensor& x, int64_t axis, qmm_tensor* t)
{
    const int64_t d = x.dim();
    if (!x.is_cuda() || x.layout() != at::kStrided || (d != 2 && d != 3) || (axis != 0 && axis != 1) || !dtype_of(x, &t->dtype)) return false;
    t->contract_axis = (int32_t)axis;
    t->rows = x.size(d - 2); t->cols = x.size(d - 1);
    t->batch = d == 3 ? x.size(0) : 1;
    t->row_stride = x.stride(d - 2);
    t->batch_stride = d == 3 ? x.stride(0) : t->rows * t->row_stride;
    if (x.stride(d - 1) != 1 && t->cols > 1) return false;
    t->data = x.data_ptr();
    return true;
}
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }
at::Tensor empty(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) { return at::empty(shape, like.options().dtype(type).requires_grad(false)); }

// args: x, contract_axis, fmt, per_channel, batch_groups, mode, seed, offset, batch_inner.  0: not the plain case; else the status
// is in *st and, if it is QMM_OK, codes and delta are filled and g is the granularity.
bool scale_quantize_call(PyObject* const* args, at::Tensor* codes, at::Tensor* delta, qmm_granularity* g, int64_t* fmt, qmm_status* st)
{
    int64_t axis, channel, groups, mode, inner;
    if (!plain(args[0]) || modes_active() || !number(args[1], &axis) || !number(args[2], fmt) || !number(args[3], &channel) ||
        !number(args[4], &groups) || !number(args[5], &mode) || !PyLong_Check(args[6]) || !PyLong_Check(args[7]) || !number(args[8], &inner))
        return false;
    const at::Tensor& x = THPVariable_Unpack(args[0]);
    qmm_tensor t;
    if (channel < 0 || channel > 1 || groups < 1 || groups > 0x7FFFFFFF || inner < 0 || inner > 0x7FFFFFFF || *fmt < 0 || *fmt > 3 || mode < 0 || mode > 1 ||
        !describe(x, axis, &t)) return false;
    const uint64_t seed = PyLong_AsUnsignedLongLongMask(args[6]), offset = PyLong_AsUnsignedLongLongMask(args[7]);
    if (PyErr_Occurred()) { PyErr_Clear(); return false; }
    *g = qmm_granularity{(int32_t)channel, (int32_t)inner, groups};
    const int64_t nc = axis == 1 ? t.rows : t.cols, kc = axis == 1 ? t.cols : t.rows;
    Unlocked unlocked;
    *delta = empty({groups * (channel ? nc : 1)}, at::kFloat, x);
    *codes = empty({t.batch, nc, kc}, at::kByte, x);
    const size_t bytes = qmm_scale_quantize_workspace_size(&t, g);
    at::Tensor ws;
    if (bytes) ws = empty({(int64_t)bytes}, at::kByte, x);
    *st = qmm_scale_quantize(&t, (qmm_format)*fmt, g, (qmm_round)mode, seed, offset, static_cast<float*>(delta->data_ptr()),
                             static_cast<uint8_t*>(codes->data_ptr()), bytes ? ws.data_ptr() : nullptr, bytes, stream());
    return true;
}

PyObject* scale_quantize(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    at::Tensor codes, delta;
    qmm_granularity g; int64_t fmt; qmm_status st;
    if (n != 9 || !scale_quantize_call(args, &codes, &delta, &g, &fmt, &st)) Py_RETURN_NONE;
    if (st != QMM_OK) return PyLong_FromLong(st);
    PyObject* c = THPVariable_Wrap(std::move(codes));
    PyObject* d = THPVariable_Wrap(std::move(delta));
    if (!c || !d) { Py_XDECREF(c); Py_XDECREF(d); return nullptr; }
    PyObject* r = PyTuple_Pack(2, c, d);
    Py_DECREF(c); Py_DECREF(d);
    return r;
    END_HANDLE_TH_ERRORS
}

// A filled Operand that keeps its tensors alive.
PyObject* make_operand(const qmm_operand& value, PyObject* data, PyObject* delta)
{
    PyObject* op = PyObject_CallObject(reinterpret_cast<PyObject*>(operand_type), nullptr);
    if (!op) return nullptr;
    Py_buffer view;
    if (PyObject_GetBuffer(op, &view, PyBUF_WRITABLE) != 0) { Py_DECREF(op); return nullptr; }
    const bool fits = view.len == (Py_ssize_t)sizeof(qmm_operand);
    if (fits) memcpy(view.buf, &value, sizeof(qmm_operand));
    PyBuffer_Release(&view);
    PyObject* keep = fits ? PyTuple_Pack(2, data, delta) : nullptr;
    if (!keep || PyObject_SetAttrString(op, "_keep", keep) != 0) {
        if (!fits) PyErr_SetString(PyExc_TypeError, "Operand is not a qmm_operand");
        Py_XDECREF(keep); Py_DECREF(op);
        return nullptr;
    }
    Py_DECREF(keep);
    return op;
}

PyObject* quantized_operand(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    at::Tensor codes, delta;
    qmm_granularity g; int64_t fmt; qmm_status st;
    if (n != 9 || !operand_type || !scale_quantize_call(args, &codes, &delta, &g, &fmt, &st)) Py_RETURN_NONE;
    if (st != QMM_OK) return PyLong_FromLong(st);
    const qmm_operand value{codes.data_ptr(), (int32_t)fmt, 1, static_cast<const float*>(delta.data_ptr()), g};
    PyObject* c = THPVariable_Wrap(std::move(codes));
    PyObject* d = THPVariable_Wrap(std::move(delta));
    PyObject* op = c && d ? make_operand(value, c, d) : nullptr;
    PyObject* pair = op ? PyTuple_Pack(2, c, op) : nullptr;
    PyObject* r = pair ? PyTuple_Pack(2, pair, d) : nullptr;
    Py_XDECREF(c); Py_XDECREF(d); Py_XDECREF(op); Py_XDECREF(pair);
    return r;
    END_HANDLE_TH_ERRORS
}

bool operand_of(PyObject* pair, const at::Tensor** data, qmm_operand* op)
{
    if (!PyTuple_CheckExact(pair) || PyTuple_GET_SIZE(pair) != 2 || !plain(PyTuple_GET_ITEM(pair, 0)) || Py_TYPE(PyTuple_GET_ITEM(pair, 1)) != operand_type)
        return false;
    *data = &THPVariable_Unpack(PyTuple_GET_ITEM(pair, 0));
    Py_buffer view;
    if (PyObject_GetBuffer(PyTuple_GET_ITEM(pair, 1), &view, PyBUF_SIMPLE) != 0) { PyErr_Clear(); return false; }
    const bool fits = view.len == (Py_ssize_t)sizeof(qmm_operand);
    if (fits) memcpy(op, view.buf, sizeof(qmm_operand));
    PyBuffer_Release(&view);
    return fits;
}

// args: a, b, out_dtype, out (or None)
PyObject* gemm(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *ta, *tb;
    qmm_operand oa, ob;
    if (n != 4 || !operand_type || modes_active() || !operand_of(args[0], &ta, &oa) || !operand_of(args[1], &tb, &ob)) Py_RETURN_NONE;
    const int64_t d = ta->dim();
    if (!ta->is_cuda() || (d != 2 && d != 3) || tb->dim() != d) Py_RETURN_NONE;
    const int64_t batch = d == 3 ? ta->size(0) : 1, M = ta->size(d - 2), K = ta->size(d - 1), N = tb->size(d - 2);
    if ((d == 3 && tb->size(0) != batch) || tb->size(d - 1) != K) Py_RETURN_NONE;
    at::Tensor y;
    at::ScalarType type;
    const bool given = args[3] != Py_None;
    if (given) {
        if (!plain(args[3])) Py_RETURN_NONE;
        y = THPVariable_Unpack(args[3]);
        type = y.scalar_type();
    } else {
        if (!THPDtype_Check(args[2])) Py_RETURN_NONE;
        type = reinterpret_cast<THPDtype*>(args[2])->scalar_type;
    }
    if (type != at::kBFloat16 && type != at::kFloat) Py_RETURN_NONE;
    qmm_status st;
    {
        Unlocked unlocked;
        if (!given) y = empty({batch, M, N}, type, *ta);
        const size_t bytes = qmm_gemm_workspace_size(&oa, &ob, batch, M, N, K);
        at::Tensor ws;
        if (bytes) ws = empty({(int64_t)bytes}, at::kByte, *ta);
        st = qmm_gemm(&oa, &ob, batch, M, N, K, y.data_ptr(), type == at::kBFloat16 ? QMM_DT_BF16 : QMM_DT_F32, nullptr,
                      bytes ? ws.data_ptr() : nullptr, bytes, stream());
    }
    if (st != QMM_OK) return PyLong_FromLong(st);
    if (given) { Py_INCREF(args[3]); return args[3]; }
    return THPVariable_Wrap(std::move(y));
    END_HANDLE_TH_ERRORS
}

// args: y, y_ref, denom, out, workspace (the last three or None)
PyObject* metric(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 5 || modes_active() || !plain(args[0]) || !plain(args[1])) Py_RETURN_NONE;
    for (int i = 2; i < 5; ++i)
        if (args[i] != Py_None && !plain(args[i])) Py_RETURN_NONE;
    const at::Tensor &y = THPVariable_Unpack(args[0]), &ref = THPVariable_Unpack(args[1]);
    int32_t type;
    const int64_t count = y.numel();
    if (!y.is_cuda() || !dtype_of(y, &type) || !y.is_contiguous() || !ref.is_contiguous() || ref.scalar_type() != at::kFloat || ref.numel() != count)
        Py_RETURN_NONE;
    const float* denom = nullptr;
    if (args[2] != Py_None) {
        const at::Tensor& d = THPVariable_Unpack(args[2]);
        if (d.numel() != count || d.scalar_type() != at::kFloat) Py_RETURN_NONE;
        denom = static_cast<const float*>(d.data_ptr());
    }
    at::Tensor out, ws;
    if (args[3] != Py_None) out = THPVariable_Unpack(args[3]);
    if (args[4] != Py_None) ws = THPVariable_Unpack(args[4]);
    qmm_status st;
    {
        Unlocked unlocked;
        if (!out.defined()) out = empty({16}, at::kDouble, y);
        if (!ws.defined()) ws = empty({std::max<int64_t>((int64_t)qmm_metric_workspace_size(count), 16)}, at::kByte, y);
        st = qmm_metric(y.data_ptr(), (qmm_dtype)type, static_cast<const float*>(ref.data_ptr()), denom, count, static_cast<double*>(out.data_ptr()),
                        ws.data_ptr(), (size_t)ws.numel(), stream());
    }
    if (st != QMM_OK) return PyLong_FromLong(st);
    if (args[3] != Py_None) { Py_INCREF(args[3]); return args[3]; }
    return THPVariable_Wrap(std::move(out));
    END_HANDLE_TH_ERRORS
}

PyObject* setup(PyObject*, PyObject* type)
{
    if (!PyType_Check(type)) { PyErr_SetString(PyExc_TypeError, "a type"); return nullptr; }
    Py_INCREF(type);
    Py_XDECREF(reinterpret_cast<PyObject*>(operand_type));
    operand_type = reinterpret_cast<PyTypeObject*>(type);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"scale_quantize", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(scale_quantize)), METH_FASTCALL, nullptr},
    {"quantized_operand", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(quantized_operand)), METH_FASTCALL, nullptr},
    {"gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(gemm)), METH_FASTCALL, nullptr},
    {"metric", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(metric)), METH_FASTCALL, nullptr},
    {"setup", setup, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_qmm_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__qmm_host(void) { return PyModule_Create(&module); }
