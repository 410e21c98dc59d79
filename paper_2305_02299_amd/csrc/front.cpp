// _front: the calls a program repeats (forward passes, condensing, connectivity updates) from Python into libsrigl without
// ctypes.  A call on a small layer runs 3-4 us on the GPU; through ctypes its 17 arguments, the stream object and the output
// allocation cost 10 us of host time, which was then what a stream of such calls ran at.  Here an argument is a pointer read
// out of the tensor object, the stream comes from the thread's current one, and the output is allocated next to the launch.
// Same names, argument order and checks as binding.py; all arithmetic stays in libsrigl.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdio>

#include <ATen/core/Tensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "pinned_answer.h"
#include "srigl.h"

namespace {

PyObject* g_error = nullptr;   // SriglError(status, where)

struct Failed {};              // a Python exception is set

[[noreturn]] void fail(PyObject* type, const char* what) {
    PyErr_SetString(type, what);
    throw Failed{};
}

void check(srigl_status st, const char* where) {
    if (st == SRIGL_OK) return;
    PyObject* e = PyObject_CallFunction(g_error, "is", (int)st, where);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    throw Failed{};
}

// The tensor in an argument, or null for None.
const at::Tensor* tensor(PyObject* o) {
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "a tensor is expected");
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) fail(PyExc_AssertionError, "device-resident contiguous tensors only");
    return &t;
}
template <typename T = void>
T* pointer(PyObject* o) {
    const at::Tensor* t = tensor(o);
    return t ? static_cast<T*>(t->data_ptr()) : nullptr;
}
size_t bytes_of(PyObject* o) {
    const at::Tensor* t = tensor(o);
    return t ? (size_t)t->numel() * t->element_size() : 0;
}
// What int() accepts (a float of a schedule, a numpy number, a tensor of one element), as in the ctypes calls.
long long integer(PyObject* o) {
    long long v = PyLong_AsLongLong(o);
    if (v != -1 || !PyErr_Occurred()) return v;
    if (!PyErr_ExceptionMatches(PyExc_TypeError)) throw Failed{};
    PyErr_Clear();
    PyObject* made = PyNumber_Long(o);
    if (!made) throw Failed{};
    v = PyLong_AsLongLong(made);
    Py_DECREF(made);
    if (v == -1 && PyErr_Occurred()) throw Failed{};
    return v;
}
int32_t int32(PyObject* o) {
    const long long v = integer(o);
    if (v != (int32_t)v) fail(PyExc_OverflowError, "a 32-bit integer is expected");
    return (int32_t)v;
}
// 16-bit containers carry bf16 bit patterns
srigl_dtype dtype_of(const at::Tensor& t) {
    const auto s = t.scalar_type();
    if (s == at::kFloat) return SRIGL_F32;
    if (s == at::kBFloat16 || s == at::kUInt16 || s == at::kShort) return SRIGL_BF16;
    fail(PyExc_TypeError, "unsupported element type");
}
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

void need(Py_ssize_t n, Py_ssize_t want) {
    if (n != want) fail(PyExc_TypeError, "wrong number of arguments");
}

// A new tensor where `like` is, straight from the caching allocator (the dispatcher's way costs another 0.3 us).
at::Tensor fresh(at::IntArrayRef size, at::ScalarType type, const at::Tensor& like) {
    return at::Tensor(at::detail::empty_cuda(size, type, like.device(), std::nullopt));
}

// The tensor y names, or a new one [B, d_out] fp32 where x is; `out` becomes the reference to return.
float* output(PyObject* y, const at::Tensor& x, int32_t B, int32_t d_out, PyObject*& out) {
    if (y != Py_None) {
        float* p = pointer<float>(y);
        Py_INCREF(y);
        out = y;
        return p;
    }
    at::Tensor t = fresh({B, d_out}, at::kFloat, x);
    float* p = static_cast<float*>(t.data_ptr());
    out = THPVariable_Wrap(std::move(t));
    if (!out) throw Failed{};
    return p;
}

// The rows of x, which must be [rows, d_in].
int32_t rows_of(const at::Tensor& x, int32_t d_in) {
    if (x.dim() != 2 || x.size(1) != d_in) fail(PyExc_AssertionError, "x is [batch, d_in]");
    if (x.size(0) > INT32_MAX) fail(PyExc_OverflowError, "batch");
    return (int32_t)x.size(0);
}

// The interpreter's lock released, and taken again at the block's end however it is left.
struct Unlocked {
    PyThreadState* const state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked&) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};

template <typename Body>
PyObject* guarded(Body body) {
    PyObject* out = nullptr;
    try {
        body(out);
        return out;
    } catch (const Failed&) {
    } catch (const std::exception& e) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    Py_XDECREF(out);
    return nullptr;
}

PyObject* set_error(PyObject*, PyObject* type) {
    Py_XDECREF(g_error);
    Py_INCREF(type);
    g_error = type;
    Py_RETURN_NONE;
}

// Device memory for the blocked copy of a call's terms, or an undefined tensor where there is none to be had (the call then takes the
// form that needs none) or where the current stream is another device's.  Given back to the allocator when the call returns, in the
// order of the current stream, on which the call has put its work.
at::Tensor scratch(size_t bytes, const at::Tensor& like) {
    if (like.device().index() != c10::hip::getCurrentHIPStream().device_index()) return at::Tensor();
    try {
        return fresh({(int64_t)bytes}, at::kByte, like);
    } catch (const c10::OutOfMemoryError&) {
        return at::Tensor();
    }
}

// linear_fwd(x, B, d_in, W_c, idx, active, n_active, K, bias, d_out, y, seg, packed, act[, blocked]) -> y
// B None: the rows of x, which must be [rows, d_in]; y None: allocated; idx in a 16-bit container: the narrow-index call.
// blocked: the call may take the matrix cores, from this copy of the terms, or with None from one that it makes for itself, in the same
// stream and from what the arrays hold then.  Nothing is kept: 4096 -> 16384 (13108 rows stored, K = 205) at batch 2048 pays 10 us of
// 210 for it, and weights that changed since, in whatever way, are the weights that count.
PyObject* linear_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](PyObject*& out) {
        if (n != 15) need(n, 14);
        const at::Tensor* x = tensor(a[0]);
        const at::Tensor* W_c = tensor(a[3]);
        const at::Tensor* idx = tensor(a[4]);
        if (!x || !W_c || !idx) fail(PyExc_TypeError, "x, W_c and idx are tensors");
        const int32_t d_in = int32(a[2]), n_active = int32(a[6]), K = int32(a[7]), d_out = int32(a[9]);
        const int32_t B = a[1] == Py_None ? rows_of(*x, d_in) : int32(a[1]);
        if (B < 0 && a[10] == Py_None) fail(PyExc_ValueError, "a negative batch");
        const int32_t* active = pointer<int32_t>(a[5]);
        const float* bias = pointer<float>(a[8]);
        const uint16_t* seg = pointer<uint16_t>(a[11]);
        const void* packed = pointer(a[12]);
        const srigl_activation act = (srigl_activation)int32(a[13]);
        float* y = output(a[10], *x, B, d_out, out);
        const srigl_dtype xt = dtype_of(*x), wt = dtype_of(*W_c);
        const void *xp = x->data_ptr(), *wp = W_c->data_ptr(), *ip = idx->data_ptr();
        const bool narrow = idx->scalar_type() != at::kInt;   // (16-bit indices are read without the streaming copy)
        void* st = stream();
        srigl_status rc;
        if (n == 15 && xt == SRIGL_BF16 && wt == SRIGL_BF16 && seg) {
            const at::Tensor* copy = tensor(a[14]);
            if ((copy ? srigl_blocked_tile : srigl_blocked_tile_with_copy)(B, d_in, n_active, K, d_out) != 0) {
                const size_t bytes = srigl_blocked_bytes(n_active, K, d_in);
                if (copy && bytes_of(a[14]) < bytes) fail(PyExc_ValueError, "a blocked copy of other rows");
                const at::Tensor made = copy ? at::Tensor() : scratch(bytes, *W_c);
                void* blocked = copy ? copy->data_ptr() : made.defined() ? made.data_ptr() : nullptr;
                if (blocked) {
                    rc = SRIGL_OK;
                    Py_BEGIN_ALLOW_THREADS
                    if (!copy) rc = srigl_block_terms(wp, ip, narrow ? 16 : 32, seg, n_active, K, d_in, blocked, bytes, st);
                    if (rc == SRIGL_OK)
                        rc = srigl_blocked_linear_fwd(xp, B, d_in, blocked, wp, ip, narrow ? 16 : 32, active, n_active, K, bias, d_out, y, act, 0, st);
                    Py_END_ALLOW_THREADS
                    check(rc, "srigl_blocked_linear_fwd");
                    return;
                }
            }
        }
        Py_BEGIN_ALLOW_THREADS
        rc = narrow ? srigl_condensed_linear_fwd_idx16(xp, xt, B, d_in, wp, wt, static_cast<const uint16_t*>(ip), active, n_active, K, bias, d_out, y,
                                                       seg, act, SRIGL_FWD_AUTO, nullptr, st)
                    : srigl_condensed_linear_fwd_act(xp, xt, B, d_in, wp, wt, static_cast<const int32_t*>(ip), active, n_active, K, bias, d_out, y,
                                                     seg, packed, act, SRIGL_FWD_AUTO, nullptr, st);
        Py_END_ALLOW_THREADS
        check(rc, narrow ? "srigl_condensed_linear_fwd_idx16" : "srigl_condensed_linear_fwd");
    });
}

// structured_fwd(x, d_in, Wd, active, n_active, bias, d_out, y, workspace) -> y, in the library's tile and parts of d_in
PyObject* structured_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](PyObject*& out) {
        need(n, 9);
        const at::Tensor* x = tensor(a[0]);
        const at::Tensor* Wd = tensor(a[2]);
        if (!x || !Wd) fail(PyExc_TypeError, "x and Wd are tensors");
        const int32_t d_in = int32(a[1]), n_active = int32(a[4]), d_out = int32(a[6]);
        const int32_t B = rows_of(*x, d_in);
        const int32_t* active = pointer<int32_t>(a[3]);
        const float* bias = pointer<float>(a[5]);
        void* ws = pointer(a[8]);
        const size_t ws_bytes = bytes_of(a[8]);
        float* y = output(a[7], *x, B, d_out, out);
        const srigl_dtype xt = dtype_of(*x), wt = dtype_of(*Wd);
        const void *xp = x->data_ptr(), *wp = Wd->data_ptr();
        void* st = stream();
        srigl_status rc;
        Py_BEGIN_ALLOW_THREADS
        rc = srigl_structured_linear_fwd_split(xp, xt, B, d_in, wp, wt, active, n_active, bias, d_out, y, SRIGL_TILE_AUTO, 0, ws, ws_bytes, st);
        Py_END_ALLOW_THREADS
        check(rc, "srigl_structured_linear_fwd_split");
    });
}

// choose(x, d_in, n_active, K, d_out, W_c) -> whether the structured-only form is expected to be faster for the rows of x
PyObject* choose(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](PyObject*& out) {
        need(n, 6);
        const at::Tensor *x = tensor(a[0]), *W_c = tensor(a[5]);
        if (!x || !W_c) fail(PyExc_TypeError, "x and W_c are tensors");
        const int32_t d_in = int32(a[1]);
        const bool s = srigl_choose_representation(rows_of(*x, d_in), d_in, int32(a[2]), int32(a[3]), int32(a[4]), dtype_of(*W_c), nullptr, nullptr) ==
                       SRIGL_REPR_STRUCTURED;
        out = PyBool_FromLong(s);
    });
}

// split_bytes(x, d_in, n_active, d_out, W_c) -> workspace bytes structured_fwd needs for the rows of x
PyObject* split_bytes(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](PyObject*& out) {
        need(n, 5);
        const at::Tensor *x = tensor(a[0]), *W_c = tensor(a[4]);
        if (!x || !W_c) fail(PyExc_TypeError, "x and W_c are tensors");
        const int32_t d_in = int32(a[1]);
        size_t bytes = 0;
        check(srigl_structured_split_plan(rows_of(*x, d_in), d_in, int32(a[2]), int32(a[3]), dtype_of(*W_c), nullptr, &bytes),
              "srigl_structured_split_plan");
        out = PyLong_FromSize_t(bytes);
    });
}

// mask_update(W, mask, grad, d_out, d_in, k, K_upd, gamma_percent, budget, mask_out, W_out, workspace, report)
PyObject* mask_update(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](PyObject*& out) {
        need(n, 13);
        const float* W = pointer<float>(a[0]);
        const uint8_t* mask = pointer<uint8_t>(a[1]);
        const float* grad = pointer<float>(a[2]);
        const int32_t d_out = int32(a[3]), d_in = int32(a[4]), k = int32(a[5]), gamma = int32(a[7]);
        const int64_t K_upd = integer(a[6]), budget = integer(a[8]);
        uint8_t* mask_out = pointer<uint8_t>(a[9]);
        float* W_out = pointer<float>(a[10]);
        void* ws = pointer(a[11]);
        const size_t ws_bytes = bytes_of(a[11]);
        int64_t* report = pointer<int64_t>(a[12]);
        void* st = stream();
        srigl_status rc;
        Py_BEGIN_ALLOW_THREADS
        rc = srigl_mask_update(W, mask, grad, d_out, d_in, k, K_upd, gamma, budget, mask_out, W_out, ws, ws_bytes, report, st);
        Py_END_ALLOW_THREADS
        check(rc, "srigl_mask_update");
        Py_INCREF(Py_None);
        out = Py_None;
    });
}

// condense(W, mask, K, want_seg, want_packed) -> (n_active, W_c, idx, active, seg, packed), every array cut to the stored rows
// (active: None when no neuron is ablated).  The arrays are complete in stream order like any other result; only the number of stored rows is waited for, which a
// launch writes straight into pinned host memory (no copy launch, no stream synchronisation).  Where the library counts rows into host memory
// (srigl_condense_count_bytes) that is the first launch, and the results are allocated and the second launch is made while it runs (768 -> 3072: 12.9 us a call, 16.2
// with both launches behind the allocations and the report of the second one, as on the other layers).
PyObject* condense(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
    return guarded([&](PyObject*& out) {
        need(n_args, 5);
        const at::Tensor *W = tensor(a[0]), *mask = tensor(a[1]);
        if (!W || !mask || mask->dim() != 2) fail(PyExc_TypeError, "W and a two-dimensional mask");
        if (mask->size(0) > INT32_MAX || mask->size(1) > INT32_MAX) fail(PyExc_OverflowError, "mask");
        const int32_t d_out = (int32_t)mask->size(0), d_in = (int32_t)mask->size(1), K = int32(a[2]);
        const bool want_seg = PyObject_IsTrue(a[3]) == 1, want_packed = PyObject_IsTrue(a[4]) == 1;
        const srigl_dtype wt = dtype_of(*W);
        const c10::hip::HIPStream st = c10::hip::getCurrentHIPStream();
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st.stream(), &capture) != hipSuccess || capture != hipStreamCaptureStatusNone)
            fail(PyExc_RuntimeError, "the report is waited for, which a captured stream cannot be (srigl_condense can)");
        const int64_t k = K > 0 ? K : 0;
        const size_t ws_bytes = srigl_workspace_bytes(d_out);
        at::Tensor active = fresh({d_out + (int64_t)(ws_bytes + 3) / 4}, at::kInt, *W);   // (with the workspace behind it)
        int32_t* const ws = static_cast<int32_t*>(active.data_ptr()) + d_out;
        // (from the allocator that pinned tensors come from: nothing here needs the tensor around it)
        const size_t count_bytes = srigl_condense_count_bytes(d_out, d_in);
        at::DataPtr pinned = at::globalContext().getPinnedMemoryAllocator(at::kCUDA)->allocate(std::max(count_bytes, sizeof(srigl_report)));
        void* const counts = count_bytes ? pinned.get() : nullptr;
        srigl_report* const rep = static_cast<srigl_report*>(pinned.get());   // (without counts: the second launch's report)
        constexpr int32_t kPending = -7;
        if (!counts) __atomic_store_n(&rep->status, kPending, __ATOMIC_RELEASE);
        at::Tensor W_c, idx, seg, packed;
        const size_t packed_bytes = srigl_packed_bytes(d_out, K, d_in, wt);
        const void* const wp = W->data_ptr();
        const uint8_t* const mp = static_cast<const uint8_t*>(mask->data_ptr());
        srigl_report report{};
        int32_t from = 0;
        srigl_status rc = SRIGL_OK;
        bool answered = false;
        {
            const Unlocked unlocked;   // (a launch on a stream whose queue is full waits for room in it)
            // Whatever happens from here on, what the launches still write into the pinned memory is waited for before it is given back.
            srigl::PinnedAnswer answer(
                [&] {
                    if (counts) return srigl_condense_counted(counts, d_out, K, d_out, &from, &report) != 0;
                    if (__atomic_load_n(&rep->status, __ATOMIC_ACQUIRE) == kPending) return false;
                    report = *rep;
                    return true;
                },
                [&] {
                    try {
                        return st.query() ? srigl::StreamState::kIdle : srigl::StreamState::kBusy;
                    } catch (...) {
                        return srigl::StreamState::kUnknown;
                    }
                },
                [&] { pinned.release_context(); });
            auto allocate = [&] {
                W_c = fresh({d_out, k}, W->scalar_type(), *W);
                idx = fresh({d_out, k}, at::kInt, *W);
                if (want_seg) seg = fresh({d_out, srigl_seg_stride(d_in)}, at::kShort, *W);
                if (want_packed) packed = fresh({(int64_t)(packed_bytes > 16 ? packed_bytes : 16)}, at::kByte, *W);
            };
            auto write = [&](auto call) {
                return call(wp, wt, mp, d_out, d_in, K, d_out, W_c.data_ptr(), static_cast<int32_t*>(idx.data_ptr()), static_cast<int32_t*>(active.data_ptr()),
                            want_seg ? static_cast<uint16_t*>(seg.data_ptr()) : nullptr, want_packed ? packed.data_ptr() : nullptr,
                            want_packed ? (size_t)packed.numel() : 0, ws, ws_bytes, counts ? nullptr : rep, st.stream());
            };
            if (counts) {
                rc = answer.launch([&] { return srigl_condense_count(mp, d_out, d_in, K, ws, ws_bytes, counts, count_bytes, st.stream()); });
                if (rc == SRIGL_OK) allocate();
                if (rc == SRIGL_OK) rc = write(srigl_condense_write);
            } else {
                allocate();
                rc = answer.launch([&] { return write(srigl_condense); });
            }
            answered = answer.wait();
        }
        check(rc, "srigl_condense");
        if (!answered) check(SRIGL_ERR_HIP, "srigl_condense");
        if (report.status != SRIGL_OK) {
            char where[64];
            snprintf(where, sizeof(where), "srigl_condense (first bad row %d)", (int)report.first_bad_row);
            check((srigl_status)report.status, where);
        }
        const int64_t n = report.n_active;
        auto cut = [&](at::Tensor& t, int64_t rows) { return THPVariable_Wrap(rows == t.size(0) ? std::move(t) : t.narrow(0, 0, rows)); };
        auto none = [] { Py_INCREF(Py_None); return Py_None; };
        PyObject* parts[5] = {cut(W_c, n), cut(idx, n), n == d_out ? none() : cut(active, n), want_seg ? cut(seg, n) : none(),
                              want_packed && n && K ? cut(packed, (int64_t)srigl_packed_bytes((int32_t)n, K, d_in, wt)) : none()};
        out = Py_BuildValue("(LNNNNN)", (long long)n, parts[0], parts[1], parts[2], parts[3], parts[4]);
        if (!out) throw Failed{};
    });
}

PyMethodDef methods[] = {
    {"set_error", set_error, METH_O, "the exception type of a failed call"},
    {"linear_fwd", (PyCFunction)(void (*)(void))linear_fwd, METH_FASTCALL, "srigl_condensed_linear_fwd"},
    {"structured_fwd", (PyCFunction)(void (*)(void))structured_fwd, METH_FASTCALL, "srigl_structured_linear_fwd_split"},
    {"choose", (PyCFunction)(void (*)(void))choose, METH_FASTCALL, "srigl_choose_representation"},
    {"split_bytes", (PyCFunction)(void (*)(void))split_bytes, METH_FASTCALL, "srigl_structured_split_plan"},
    {"condense", (PyCFunction)(void (*)(void))condense, METH_FASTCALL, "srigl_condense into new tensors"},
    {"mask_update", (PyCFunction)(void (*)(void))mask_update, METH_FASTCALL, "srigl_mask_update"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_front", "calls into libsrigl", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__front() { return PyModule_Create(&module); }
