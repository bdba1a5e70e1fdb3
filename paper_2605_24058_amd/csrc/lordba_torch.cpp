// The calls of the Python binding on torch tensors, in C++: reading the tensors, allocating the outputs and calling the C
// interface (include/lordba.h).  A call of one token took 7.4 us on the host through Python's attribute reads and ctypes (2.0 for the
// checks, 1.2 for the output), while its kernel runs for 4.3; so it takes 4.9, and a small training step 31 instead of 47.
//
// Every function takes the arguments of the binding's function of that name and returns what that returns; an int, the library's
// status, where the call failed; or None where the arguments are not the plain case: ordinary CUDA tensors, contiguous, of the
// expected types and shapes.  The binding then goes its own way, which is also where exceptions come from.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/PyInterpreter.h>
#include <torch/csrc/autograd/python_variable.h>

#include "lordba.h"

namespace {

constexpr at::ScalarType kF16 = at::kHalf, kF32 = at::kFloat, kI32 = at::kInt;

// The tensor behind `o`, or nullptr if it is not a plain contiguous CUDA tensor of this type (subclasses, wrapped tensors without
// storage and the like are not).
const at::Tensor* plain(PyObject* o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || t.scalar_type() != type || !t.is_contiguous())
        return nullptr;
    return &t;
}

template <typename T>
T* ptr(const at::Tensor* t) { return t ? static_cast<T*>(t->data_ptr()) : nullptr; }
template <typename T>
T* ptr(const at::Tensor& t) { return static_cast<T*>(t.data_ptr()); }

int64_t words(int64_t rows, int64_t cols) { return (rows * cols + 31) / 32; }

bool shaped(const at::Tensor* t, std::initializer_list<int64_t> s) { return t->sizes() == at::IntArrayRef(s); }

// the stream to enqueue on: a handle, or (None) torch's current stream of the tensor's device
bool stream_of(PyObject* o, const at::Tensor* t, void** out) {
    if (o == Py_None) {
        *out = c10::hip::getCurrentHIPStream(t->get_device()).stream();
        return true;
    }
    if (!PyLong_CheckExact(o)) return false;
    *out = PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}

// Nobody watches or replaces torch's own functions (a mode that does would miss the allocations made here, or hand out tensors that have
// no memory).  Default devices are modes too (torch.set_default_device, `with torch.device(...)`) and concern nothing here: every
// allocation names its device.
PyObject* device_mode = nullptr;   // torch.utils._device.DeviceContext
bool unwatched() {
    for (int64_t i = at::impl::PythonTorchFunctionTLS::stack_len() - 1; i >= 0; --i) {
        PyObject* mode = at::impl::PythonTorchFunctionTLS::get_stack_at(i)->ptr(getPyInterpreter());
        if (reinterpret_cast<PyObject*>(Py_TYPE(mode)) != device_mode) return false;
    }
    return !c10::impl::TorchDispatchModeTLS::any_modes_set();
}

// A number of the kind that float() takes as it is: a float or an int (others go the binding's own way).
bool number(PyObject* o, float* out) {
    if (!PyFloat_Check(o) && !PyLong_Check(o)) return false;
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) { PyErr_Clear(); return false; }
    *out = static_cast<float>(v);
    return true;
}

at::Tensor empty(const at::Tensor* like, at::ScalarType type, std::initializer_list<int64_t> s) {
    return at::empty(at::IntArrayRef(s), at::TensorOptions().dtype(type).device(like->device()));
}

#define NEED(cond) do { if (!(cond)) Py_RETURN_NONE; } while (0)

// y_out: an argument or None; false: not the plain case
bool output_like(PyObject* o, const at::Tensor* y_base, at::Tensor* out) {
    if (o == Py_None) { *out = at::empty_like(*y_base); return true; }
    const at::Tensor* t = plain(o, kF16);
    if (!t || t->sizes() != y_base->sizes()) return false;
    *out = *t;
    return true;
}

struct Forward {   // what the four forward calls share: x, packedA, packedB, s_in, s_rank, s_out, y_base
    const at::Tensor *x, *pA, *pB, *si, *sr, *so, *yb;
    int64_t T, d_in, d_out;
    bool read(PyObject* const* a, PyObject* y_base) {
        x = plain(a[0], kF16), pA = plain(a[1], kI32), pB = plain(a[2], kI32);
        si = plain(a[3], kF16), sr = plain(a[4], kF16), so = plain(a[5], kF16), yb = plain(y_base, kF16);
        if (!x || !pA || !pB || !si || !sr || !so || !yb || x->dim() != 2 || yb->dim() != 2 || x->size(0) != yb->size(0)) return false;
        T = x->size(0), d_in = x->size(1), d_out = yb->size(1);
        return true;
    }
    bool single(int64_t* r) const {   // one adapter, one envelope
        *r = sr->numel();
        return si->numel() == d_in && so->numel() == d_out && pA->numel() == words(*r, d_in) && pB->numel() == words(d_out, *r);
    }
    bool multi(int64_t* ell, int64_t* r) const {
        if (si->dim() != 2 || sr->dim() != 2 || so->dim() != 2) return false;
        *ell = sr->size(0), *r = sr->size(1);
        return shaped(si, {*ell, d_in}) && shaped(so, {*ell, d_out}) && pA->numel() == words(*r, d_in) && pB->numel() == words(d_out, *r);
    }
};

PyObject* result(const at::Tensor& t, int st) { return st == LORDBA_OK ? THPVariable_Wrap(t) : PyLong_FromLong(st); }

// f(a...) without the interpreter's lock.  The arguments are evaluated while it is held: a tensor may refuse its pointer, and an
// exception that passes must find the lock.
struct Unlocked {
    PyThreadState* const state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};
template <class F, class... A>
int unlocked(F* f, A... a) {
    Unlocked here;
    return f(a...);
}

// (x, packedA, packedB, s_in, s_rank, s_out, y_base, y_out, stream)
PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Forward f;
    int64_t r;
    void* st;
    at::Tensor y;
    NEED(n == 9 && unwatched() && f.read(a, a[6]) && f.single(&r) && stream_of(a[8], f.x, &st) && output_like(a[7], f.yb, &y));
    const int rc = unlocked(lordba_forward, ptr<void>(f.x), ptr<uint32_t>(f.pA), ptr<uint32_t>(f.pB), ptr<void>(f.si), ptr<void>(f.sr),
                            ptr<void>(f.so), ptr<void>(f.yb), ptr<void>(y), f.T, f.d_in, f.d_out, r, st);
    return result(y, rc);
    END_HANDLE_TH_ERRORS
}

PyObject* forward_multi(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Forward f;
    int64_t r, ell;
    void* st;
    at::Tensor y;
    NEED(n == 9 && unwatched() && f.read(a, a[6]) && f.multi(&ell, &r) && stream_of(a[8], f.x, &st) && output_like(a[7], f.yb, &y));
    const int rc = unlocked(lordba_forward_multi, ptr<void>(f.x), ptr<uint32_t>(f.pA), ptr<uint32_t>(f.pB), ptr<void>(f.si),
                            ptr<void>(f.sr), ptr<void>(f.so), ptr<void>(f.yb), ptr<void>(y), f.T, f.d_in, f.d_out, r, ell, st);
    return result(y, rc);
    END_HANDLE_TH_ERRORS
}

// (x, packedA_pool, packedB_pool, s_in_pool, s_rank_pool, s_out_pool, adapter_of_row, y_base, y_out, stream)
PyObject* forward_batched(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Forward f;
    void* st;
    at::Tensor y;
    NEED(n == 10 && unwatched() && f.read(a, a[7]));
    const at::Tensor* ids = plain(a[6], kI32);
    NEED(ids && ids->numel() == f.T && f.sr->dim() == 2 && f.pA->dim() == 2 && f.pB->dim() == 2);
    const int64_t na = f.sr->size(0), r = f.sr->size(1);
    NEED(shaped(f.si, {na, f.d_in}) && shaped(f.so, {na, f.d_out}) && shaped(f.pA, {na, words(r, f.d_in)}) &&
         shaped(f.pB, {na, words(f.d_out, r)}) && stream_of(a[9], f.x, &st) && output_like(a[8], f.yb, &y));
    const int rc = unlocked(lordba_forward_batched, ptr<void>(f.x), ptr<uint32_t>(f.pA), ptr<uint32_t>(f.pB), ptr<void>(f.si),
                            ptr<void>(f.sr), ptr<void>(f.so), ptr<int32_t>(ids), ptr<void>(f.yb), ptr<void>(y), f.T, f.d_in, f.d_out, r,
                            na, st);
    return result(y, rc);
    END_HANDLE_TH_ERRORS
}

PyObject* forward_batched_multi(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Forward f;
    void* st;
    at::Tensor y;
    NEED(n == 10 && unwatched() && f.read(a, a[7]));
    const at::Tensor* ids = plain(a[6], kI32);
    NEED(ids && ids->numel() == f.T && f.sr->dim() == 3);
    const int64_t na = f.sr->size(0), ell = f.sr->size(1), r = f.sr->size(2);
    NEED(shaped(f.si, {na, ell, f.d_in}) && shaped(f.so, {na, ell, f.d_out}) && shaped(f.pA, {na, words(r, f.d_in)}) &&
         shaped(f.pB, {na, words(f.d_out, r)}) && stream_of(a[9], f.x, &st) && output_like(a[8], f.yb, &y));
    const int rc = unlocked(lordba_forward_batched_multi, ptr<void>(f.x), ptr<uint32_t>(f.pA), ptr<uint32_t>(f.pB), ptr<void>(f.si),
                            ptr<void>(f.sr), ptr<void>(f.so), ptr<int32_t>(ids), ptr<void>(f.yb), ptr<void>(y), f.T, f.d_in, f.d_out, r,
                            ell, na, st);
    return result(y, rc);
    END_HANDLE_TH_ERRORS
}

// (latentA, latentB, stream, transposed)
PyObject* pack_latents(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    NEED(n == 4 && unwatched());
    const at::Tensor *A = plain(a[0], kF32), *B = plain(a[1], kF32);
    void* st;
    NEED(A && B && A->dim() == 2 && B->dim() == 2 && A->size(0) == B->size(1) && (a[3] == Py_True || a[3] == Py_False) &&
         stream_of(a[2], A, &st));
    const int64_t r = A->size(0), d_in = A->size(1), d_out = B->size(0), wA = words(r, d_in), wB = words(d_out, r);
    at::Tensor out[4];
    for (int i = 0; i < (a[3] == Py_True ? 4 : 2); ++i) out[i] = empty(A, kI32, {i & 1 ? wB : wA});
    const int rc = unlocked(lordba_pack_latents, ptr<float>(A), ptr<float>(B), ptr<uint32_t>(out[0]), ptr<uint32_t>(out[1]),
                            out[2].defined() ? ptr<uint32_t>(out[2]) : nullptr, out[3].defined() ? ptr<uint32_t>(out[3]) : nullptr, d_in,
                            d_out, r, st);
    if (rc != LORDBA_OK) return PyLong_FromLong(rc);
    PyObject* t = PyTuple_New(4);
    for (int i = 0; t && i < 4; ++i) PyTuple_SET_ITEM(t, i, THPVariable_Wrap(out[i]));   // (an undefined tensor becomes None)
    return t;
    END_HANDLE_TH_ERRORS
}

// The training forwards: (x, packedA, packedB, s_in, s_rank, s_out, y_base, stream), outputs always new
PyObject* save_t(PyObject* const* a, Py_ssize_t n, bool many) {
    Forward f;
    int64_t r, ell = 1;
    void* st;
    NEED(n == 8 && unwatched() && f.read(a, a[6]) && (many ? f.multi(&ell, &r) : f.single(&r)) && stream_of(a[7], f.x, &st));
    const int64_t stride = (f.T + 127) / 128 * 128;
    at::Tensor t = many ? empty(f.x, kF32, {ell, r, stride}) : empty(f.x, kF32, {r, stride}), y = at::empty_like(*f.yb);
    const int rc = many ? unlocked(lordba_forward_multi_save_t, ptr<void>(f.x), ptr<uint32_t>(f.pA), ptr<uint32_t>(f.pB),
                                   ptr<void>(f.si), ptr<void>(f.sr), ptr<void>(f.so), ptr<void>(f.yb), ptr<void>(y), ptr<float>(t),
                                   stride, f.T, f.d_in, f.d_out, r, ell, st)
                        : unlocked(lordba_forward_save_t, ptr<void>(f.x), ptr<uint32_t>(f.pA), ptr<uint32_t>(f.pB), ptr<void>(f.si),
                                   ptr<void>(f.sr), ptr<void>(f.so), ptr<void>(f.yb), ptr<void>(y), ptr<float>(t), stride, f.T, f.d_in,
                                   f.d_out, r, st);
    if (rc != LORDBA_OK) return PyLong_FromLong(rc);
    PyObject* out = PyTuple_New(2);
    if (out) {
        PyTuple_SET_ITEM(out, 0, THPVariable_Wrap(y));
        PyTuple_SET_ITEM(out, 1, THPVariable_Wrap(t));
    }
    return out;
}
PyObject* forward_save_t(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    return save_t(a, n, false);
    END_HANDLE_TH_ERRORS
}
PyObject* forward_multi_save_t(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    return save_t(a, n, true);
    END_HANDLE_TH_ERRORS
}

// (x, g, packedA, packedAt, packedBt, s_in, s_rank, s_out, latentA, latentB, kappa, dx_base, workspace, stream, t_saved), outputs
// always new; the latents and dx_base may be None, and so may the workspace and t_saved
PyObject* backward_any(PyObject* const* a, Py_ssize_t n, bool many) {
    NEED(n == 15 && unwatched());
    const at::Tensor *x = plain(a[0], kF16), *g = plain(a[1], kF16), *pA = plain(a[2], kI32), *pAt = plain(a[3], kI32), *pBt = plain(a[4], kI32);
    const at::Tensor *si = plain(a[5], kF16), *sr = plain(a[6], kF16), *so = plain(a[7], kF16);
    NEED(x && g && pA && pAt && pBt && si && sr && so && x->dim() == 2 && g->dim() == 2 && x->size(0) == g->size(0));
    const int64_t T = x->size(0), d_in = x->size(1), d_out = g->size(1);
    NEED(!many || (sr->dim() == 2 && si->dim() == 2 && so->dim() == 2));
    const int64_t ell = many ? sr->size(0) : 1, r = many ? sr->size(1) : sr->numel();
    NEED(many ? shaped(si, {ell, d_in}) && shaped(so, {ell, d_out}) : si->numel() == d_in && so->numel() == d_out);
    NEED(pA->numel() == words(r, d_in) && pAt->numel() == words(r, d_in) && pBt->numel() == words(r, d_out));
    const bool lat = a[8] != Py_None;
    NEED(lat == (a[9] != Py_None));
    const at::Tensor *lA = lat ? plain(a[8], kF32) : nullptr, *lB = lat ? plain(a[9], kF32) : nullptr;
    NEED(!lat || (lA && lB && shaped(lA, {r, d_in}) && shaped(lB, {d_out, r})));
    float kappa;
    NEED(number(a[10], &kappa));
    const at::Tensor *dxb = a[11] == Py_None ? nullptr : plain(a[11], kF16), *ws = a[12] == Py_None ? nullptr : plain(a[12], at::kByte);
    const at::Tensor* ts = a[14] == Py_None ? nullptr : plain(a[14], kF32);
    NEED((dxb || a[11] == Py_None) && (ws || a[12] == Py_None) && (ts || a[14] == Py_None));
    NEED((!dxb || dxb->sizes() == x->sizes()) && (!ts || ts->dim() == (many ? 3 : 2)));
    void* st;
    NEED(stream_of(a[13], x, &st));
    at::Tensor own;
    if (!ws) {
        const int64_t need = static_cast<int64_t>(many ? lordba_backward_multi_workspace_bytes(T, d_in, d_out, r, ell)
                                                       : lordba_backward_workspace_bytes(T, d_in, d_out, r));
        own = empty(x, at::kByte, {need < 16 ? 16 : need});
        ws = &own;
    }
    at::Tensor dx, out[5];
    if (dxb) dx = at::empty_like(*dxb);
    const int64_t cols[3] = {d_in, r, d_out};
    for (int i = 0; i < 3; ++i) out[i] = many ? empty(x, kF32, {ell, cols[i]}) : empty(x, kF32, {cols[i]});
    if (lat) {
        out[3] = empty(x, kF32, {r, d_in});
        out[4] = empty(x, kF32, {d_out, r});
    }
    void* const dxp = dxb ? ptr<void>(dx) : nullptr;
    float* gp[5];
    for (int i = 0; i < 5; ++i) gp[i] = out[i].defined() ? ptr<float>(out[i]) : nullptr;
    const int64_t stride = ts ? ts->size(many ? 2 : 1) : 0;
    const int rc = many ? unlocked(lordba_backward_multi, ptr<void>(x), ptr<void>(g), ptr<uint32_t>(pA), ptr<uint32_t>(pAt),
                                   ptr<uint32_t>(pBt), ptr<void>(si), ptr<void>(sr), ptr<void>(so), ptr<float>(lA), ptr<float>(lB),
                                   kappa, ptr<float>(ts), stride, ptr<void>(dxb), dxp, gp[0], gp[1], gp[2], gp[3], gp[4], ptr<void>(ws),
                                   ws->numel(), T, d_in, d_out, r, ell, st)
                        : unlocked(lordba_backward, ptr<void>(x), ptr<void>(g), ptr<uint32_t>(pA), ptr<uint32_t>(pAt),
                                   ptr<uint32_t>(pBt), ptr<void>(si), ptr<void>(sr), ptr<void>(so), ptr<float>(lA), ptr<float>(lB),
                                   kappa, ptr<float>(ts), stride, ptr<void>(dxb), dxp, gp[0], gp[1], gp[2], gp[3], gp[4], ptr<void>(ws),
                                   ws->numel(), T, d_in, d_out, r, st);
    if (rc != LORDBA_OK) return PyLong_FromLong(rc);
    static PyObject* const names[6] = {PyUnicode_InternFromString("dx"),      PyUnicode_InternFromString("d_s_in"),
                                       PyUnicode_InternFromString("d_s_rank"), PyUnicode_InternFromString("d_s_out"),
                                       PyUnicode_InternFromString("d_latentA"), PyUnicode_InternFromString("d_latentB")};
    PyObject* d = PyDict_New();
    for (int i = 0; d && i < 6; ++i) {
        PyObject* v = THPVariable_Wrap(i == 0 ? dx : out[i - 1]);   // (None where undefined)
        if (!v || PyDict_SetItem(d, names[i], v) != 0) {
            Py_XDECREF(v);
            Py_CLEAR(d);
            break;
        }
        Py_DECREF(v);
    }
    return d;
}
PyObject* backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    return backward_any(a, n, false);
    END_HANDLE_TH_ERRORS
}
PyObject* backward_multi(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    return backward_any(a, n, true);
    END_HANDLE_TH_ERRORS
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(forward),        METHOD(forward_multi),        METHOD(forward_batched), METHOD(forward_batched_multi),
                         METHOD(pack_latents),   METHOD(forward_save_t),       METHOD(forward_multi_save_t),
                         METHOD(backward),       METHOD(backward_multi),       {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lordba_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lordba_torch() {
    if (PyObject* m = PyImport_ImportModule("torch.utils._device")) {
        device_mode = PyObject_GetAttrString(m, "DeviceContext");
        Py_DECREF(m);
    }
    PyErr_Clear();   // (a torch without it: such modes then go the binding's own way)
    return PyModule_Create(&module);
}
