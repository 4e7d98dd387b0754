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
#include <cxxabi.h>
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

// The call itself, without the GIL: takes a workspace (`own`) and launches.
int launch(void* const* table, Op op, int code, int64_t N, int64_t C, int64_t HW, void* const (&big)[3],
           float* const (&chan)[6], const float (&f)[3], at::Device dev, bool own, at::Tensor& ws) {
    if (own) {
        const size_t need =
            entry<decltype(iabn_workspace_size)>(table, kWorkspaceSize)(N, C, HW, code);
        ws = at::empty({static_cast<int64_t>(need ? need : 1)},
                       at::TensorOptions().dtype(at::kByte).device(dev));
    }
    void* const wp = ws.defined() ? ws.data_ptr() : nullptr;
    const size_t wb = ws.defined() ? ws.numel() * ws.element_size() : 0;
    void* const st = c10::hip::getCurrentHIPStream(dev.index()).stream();
    switch (op) {
        case kForwardTrain:
            return entry<decltype(iabn_forward_train)>(table, op)(
                big[0], code, chan[0], chan[1], chan[2], chan[3], chan[4], chan[5], f[0], f[1], f[2], N,
                C, HW, wp, wb, st);
        case kForwardTrainNoalloc:
            return entry<decltype(iabn_forward_train_noalloc)>(table, op)(
                big[0], code, chan[0], chan[1], chan[2], chan[3], chan[4], chan[5], f[0], f[1], f[2], N,
                C, HW, st);
        case kForwardEval:
            return entry<decltype(iabn_forward_eval)>(table, op)(
                big[0], code, chan[0], chan[1], chan[2], chan[3], f[0], f[1], N, C, HW, st);
        case kBackward:
        case kBackwardII:
            return entry<decltype(iabn_backward)>(table, op)(
                big[0], big[1], code, chan[0], chan[1], chan[2], chan[3], chan[4], f[0], f[1], N, C, HW,
                wp, wb, st);
        case kStdForward:
            return entry<decltype(iabn_std_forward_train)>(table, op)(
                big[0], big[1], code, chan[0], chan[1], chan[2], chan[3], chan[4], chan[5], f[0], f[1],
                f[2], N, C, HW, wp, wb, st);
        case kStdBackward:
            return entry<decltype(iabn_std_backward)>(table, op)(
                big[0], big[1], big[2], code, chan[0], chan[1], chan[2], chan[3], chan[4], chan[5], f[0],
                f[1], N, C, HW, wp, wb, st);
        case kCkptForward:
            return entry<decltype(iabn_ckpt_forward_train)>(table, op)(
                big[0], big[1], code, chan[0], chan[1], chan[2], chan[3], chan[4], chan[5], f[0], f[1],
                f[2], N, C, HW, wp, wb, st);
        case kCkptRecompute:
            return entry<decltype(iabn_ckpt_recompute)>(table, op)(
                big[0], big[1], code, chan[0], chan[1], f[0], N, C, HW, st);
        default:
            return entry<decltype(iabn_ckpt_backward)>(table, op)(
                big[0], big[1], code, chan[0], chan[1], chan[2], chan[3], chan[4], f[0], f[1], N, C, HW,
                wp, wb, st);
    }
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
    bool own = false;
    if (s.workspace) {
        own = args[0] == Py_None;
        if (!own) {
            if (!THPVariable_CheckExact(args[0])) return not_plain();
            ws = THPVariable_Unpack(args[0]);
            if (ws.device() != dev || !ws.is_contiguous()) return not_plain();
        }
    }

    // An allocation can wait for the device and a launch for room in the
    // queue, so other Python threads go on meanwhile.
    int rc = 0;
    PyThreadState* thread = PyEval_SaveThread();
    try {
        rc = launch(table, op, code, N, C, HW, big, chan, f, dev, own, ws);
    } catch (...) {
        PyEval_RestoreThread(thread);
        throw;
    }
    PyEval_RestoreThread(thread);
    return PyLong_FromLong(rc);
}

// call(table, op, tensors..., floats...[, workspace]) -> status, or
// NotImplemented (nothing was done).  A C++ exception before the launch (no
// memory for a workspace, a tensor without storage) is left to the Python
// path to meet again and report.
PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
    try {
        return call_checked(args, n);
    } catch (abi::__forced_unwind&) {
        throw;  // the interpreter ends this thread
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
