// The Python binding's fast path: one call from Python checks the tensors of
// an entry point, takes a workspace where none is given, finds torch's
// current stream and calls libiabn.  Marshalling only, as in __init__.py,
// which this does not replace: whatever is not the plain case (a wrong
// argument, a tensor subclass, an explicit stream) returns NotImplemented,
// and the Python function then does the same checks and reports what is
// wrong.
//
// Why native: the same checks in Python and a ctypes call of 17 arguments
// took 10-13 us per call, more than the kernels of a small layer.

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "iabn.h"

namespace {

// The entry points, in the order of the table that each call is given (the
// addresses in one loaded libiabn): see _NATIVE in __init__.py.
enum Op : long {
    kWorkspaceSize,
    kForwardTrain,
    kForwardTrainNoalloc,
    kForwardEval,
    kBackward,
    kBackwardII,
    kStdForward,
    kStdBackward,
    kCkptForward,
    kCkptRecompute,
    kCkptBackward,
    kOps
};

// What follows the table and the op in a call: activation tensors,
// per-channel tensors, floats, then a workspace (or None) if it takes one.
struct Shape {
    int big, chan, floats;
    bool workspace;
};
constexpr Shape kShapes[kOps] = {{0, 0, 0, false}, {1, 6, 3, true},  {1, 6, 3, false}, {1, 4, 2, false},
                                 {2, 5, 2, true},  {2, 5, 2, true},  {2, 6, 3, true},  {3, 6, 2, true},
                                 {2, 6, 3, true},  {2, 2, 1, false}, {2, 5, 2, true}};

PyObject* not_plain() {
    PyErr_Clear();
    Py_RETURN_NOTIMPLEMENTED;
}

int dtype_code(at::ScalarType t) {
    switch (t) {
        case at::kFloat: return IABN_F32;
        case at::kHalf: return IABN_F16;
        case at::kBFloat16: return IABN_BF16;
        default: return -1;
    }
}

template <typename Fn>
Fn* entry(void* const* table, Op op) {
    return reinterpret_cast<Fn*>(table[op]);
}

PyObject* call_checked(PyObject* const* args, Py_ssize_t n) {
    if (n < 2) return not_plain();
    void* const* table = static_cast<void* const*>(PyLong_AsVoidPtr(args[0]));
    const long opn = PyLong_AsLong(args[1]);
    if (table == nullptr || opn <= kWorkspaceSize || opn >= kOps) return not_plain();
    const Op op = static_cast<Op>(opn);
    const Shape& s = kShapes[op];
    if (n != 2 + s.big + s.chan + s.floats + (s.workspace ? 1 : 0)) return not_plain();
    args += 2;

    void* big[3];
    int64_t N = 0, C = 0, HW = 1;
    int code = -1;
    at::Device dev(at::kCPU);
    for (int i = 0; i < s.big; ++i) {
        if (!THPVariable_CheckExact(args[i])) return not_plain();
        const at::Tensor& t = THPVariable_Unpack(args[i]);
        if (t.dim() < 2 || !t.is_cuda() || !t.is_contiguous()) return not_plain();
        if (i == 0) {
            N = t.size(0);
            C = t.size(1);
            for (int64_t d = 2; d < t.dim(); ++d) HW *= t.size(d);
            code = dtype_code(t.scalar_type());
            dev = t.device();
            if (code < 0) return not_plain();
        } else {
            int64_t hw = 1;
            for (int64_t d = 2; d < t.dim(); ++d) hw *= t.size(d);
            if (t.size(0) != N || t.size(1) != C || hw != HW || dtype_code(t.scalar_type()) != code ||
                t.device() != dev)
                return not_plain();
        }
        big[i] = t.data_ptr();
    }
    args += s.big;
    float* chan[6];
    for (int i = 0; i < s.chan; ++i) {
        if (!THPVariable_CheckExact(args[i])) return not_plain();
        const at::Tensor& t = THPVariable_Unpack(args[i]);
        if (t.scalar_type() != at::kFloat || !t.is_contiguous() || t.numel() != C || t.device() != dev)
            return not_plain();
        chan[i] = static_cast<float*>(t.data_ptr());
    }
    args += s.chan;
    float f[3];
    for (int i = 0; i < s.floats; ++i) {
        const double v = PyFloat_Check(args[i]) || PyLong_Check(args[i]) ? PyFloat_AsDouble(args[i]) : -1.0;
        if (PyErr_Occurred() || !(PyFloat_Check(args[i]) || PyLong_Check(args[i]))) return not_plain();
        f[i] = static_cast<float>(v);
    }
    args += s.floats;
    at::Tensor ws;
    void* wp = nullptr;
    size_t wb = 0;
    if (s.workspace) {
        if (args[0] == Py_None) {
            const size_t need =
                entry<decltype(iabn_workspace_size)>(table, kWorkspaceSize)(N, C, HW, code);
            ws = at::empty({static_cast<int64_t>(need ? need : 1)},
                           at::TensorOptions().dtype(at::kByte).device(dev));
        } else {
            if (!THPVariable_CheckExact(args[0])) return not_plain();
            ws = THPVariable_Unpack(args[0]);
            if (ws.device() != dev || !ws.is_contiguous()) return not_plain();
        }
        wp = ws.data_ptr();
        wb = ws.numel() * ws.element_size();
    }
    void* st = c10::hip::getCurrentHIPStream(dev.index()).stream();

    int rc = 0;
    Py_BEGIN_ALLOW_THREADS;  // a launch can wait for room in the queue
    switch (op) {
        case kForwardTrain:
            rc = entry<decltype(iabn_forward_train)>(table, op)(
                big[0], code, chan[0], chan[1], chan[2], chan[3], chan[4], chan[5], f[0], f[1], f[2], N,
                C, HW, wp, wb, st);
            break;
        case kForwardTrainNoalloc:
            rc = entry<decltype(iabn_forward_train_noalloc)>(table, op)(
                big[0], code, chan[0], chan[1], chan[2], chan[3], chan[4], chan[5], f[0], f[1], f[2], N,
                C, HW, st);
            break;
        case kForwardEval:
            rc = entry<decltype(iabn_forward_eval)>(table, op)(big[0], code, chan[0], chan[1], chan[2],
                                                               chan[3], f[0], f[1], N, C, HW, st);
            break;
        case kBackward:
        case kBackwardII:
            rc = entry<decltype(iabn_backward)>(table, op)(big[0], big[1], code, chan[0], chan[1],
                                                           chan[2], chan[3], chan[4], f[0], f[1], N, C,
                                                           HW, wp, wb, st);
            break;
        case kStdForward:
            rc = entry<decltype(iabn_std_forward_train)>(table, op)(
                big[0], big[1], code, chan[0], chan[1], chan[2], chan[3], chan[4], chan[5], f[0], f[1],
                f[2], N, C, HW, wp, wb, st);
            break;
        case kStdBackward:
            rc = entry<decltype(iabn_std_backward)>(table, op)(
                big[0], big[1], big[2], code, chan[0], chan[1], chan[2], chan[3], chan[4], chan[5], f[0],
                f[1], N, C, HW, wp, wb, st);
            break;
        case kCkptForward:
            rc = entry<decltype(iabn_ckpt_forward_train)>(table, op)(
                big[0], big[1], code, chan[0], chan[1], chan[2], chan[3], chan[4], chan[5], f[0], f[1],
                f[2], N, C, HW, wp, wb, st);
            break;
        case kCkptRecompute:
            rc = entry<decltype(iabn_ckpt_recompute)>(table, op)(big[0], big[1], code, chan[0], chan[1],
                                                                 f[0], N, C, HW, st);
            break;
        default:
            rc = entry<decltype(iabn_ckpt_backward)>(table, op)(big[0], big[1], code, chan[0], chan[1],
                                                                chan[2], chan[3], chan[4], f[0], f[1], N,
                                                                C, HW, wp, wb, st);
    }
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(rc);
}

// call(table, op, tensors..., floats...[, workspace]) -> status, or
// NotImplemented (nothing was done).  A C++ exception before the launch (no
// memory for a workspace, a tensor without storage) is left to the Python
// path to meet again and report.
PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
    try {
        return call_checked(args, n);
    } catch (...) {
        return not_plain();
    }
}

PyMethodDef methods[] = {
    {"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call)), METH_FASTCALL,
     "call(table, op, tensors..., floats...[, workspace]) -> status or NotImplemented"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods,
                      nullptr,               nullptr,    nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
