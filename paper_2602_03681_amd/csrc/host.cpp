// Host path of the calls that are made once per generated token (and of the plain forward): checks, output allocation
// and the call into libnats.so without a trip through Python per argument.
//
// The kernels of a step at small batches take 6 to 8 us; checking fifteen tensors and filling a ctypes call in Python took 12.5
// us per step, which a generation loop then waited for.  The functions here take the arguments of the Python functions
// of the same names by position and return
//   the output tensor   the call was made,
//   an int              it was made and refused: the library's status (its message is in nats_last_error),
//   None                an argument is not what this path takes (a wrong shape, a CPU tensor, a subclass, ...): the Python
//                       function then runs its own checks, which name what is wrong.
// A workspace that the caller did not give is allocated for the call where the step gains by it (see wants_workspace),
// from torch's caching allocator like the output, ordered on the current stream; not while the stream is being captured, where
// torch may have no pool to take it from.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>

#include "nats.h"

namespace {

struct NotTaken {};   // thrown where an argument is not what the fast path takes

const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_CheckExact(o)) throw NotTaken();
    return THPVariable_Unpack(o);
}

void* pointer(const at::Tensor& t, at::ScalarType dt, std::initializer_list<int64_t> shape) {
    if (!t.is_cuda() || t.scalar_type() != dt || t.layout() != at::kStrided ||
        t.sizes() != at::IntArrayRef(shape.begin(), shape.size()) || !t.is_contiguous())
        throw NotTaken();
    return t.data_ptr();
}

void* pointer(PyObject* o, at::ScalarType dt, std::initializer_list<int64_t> shape) { return pointer(tensor(o), dt, shape); }

void* optional(PyObject* o, at::ScalarType dt, std::initializer_list<int64_t> shape) {
    return o == Py_None ? nullptr : pointer(o, dt, shape);
}

double number(PyObject* o) {
    const double x = PyFloat_Check(o) ? PyFloat_AS_DOUBLE(o) : PyFloat_AsDouble(o);
    if (x == -1.0 && PyErr_Occurred()) { PyErr_Clear(); throw NotTaken(); }
    return x;
}

int integer(PyObject* o) {
    const long x = PyLong_AsLong(o);
    if ((x == -1 && PyErr_Occurred()) || x != (int)x) { PyErr_Clear(); throw NotTaken(); }
    return (int)x;
}

int dtype_code(at::ScalarType dt) {
    if (dt == at::kFloat) return NATS_F32;
    if (dt == at::kBFloat16) return NATS_BF16;
    throw NotTaken();
}

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// (an error, as for the null stream beside a capture of another one, counts as capturing)
bool capturing() {
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c10::hip::getCurrentHIPStream().stream(), &s) == hipSuccess) return s != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// Whether a step without a workspace of the caller's gets one: with few (batch, head) pairs one block per pair leaves the
// chip idle.  Measured (bf16, us per step, one block against blocks of 64 rows and a second kernel):
//   d 128, 16 pairs: 64 rows 6.5 / 6.3, 256 rows 8.0 / 6.6, 1000 rows 13.0 / 7.2, 2048 rows 19.6 / 9.0;
//   96 pairs, lengths spread evenly up to the figure: 256 rows 8.7 / 8.2, 1000 rows 14.9 / 10.6, 2048 rows 22.2 / 16.8;
//   192 pairs: 256 rows 10.8 / 11.1 .. 12.6, 1000 rows 19.6 / 17.8 (all equal: 23.4 / 23.5);
//   d 64, 16 pairs: 64 rows 5.1 / 6.1, 256 rows 5.8 / 6.3, 1000 rows 8.5 / 6.7, 2048 rows 12.1 / 7.6.
// The lengths are on the device; what is known here is the capacity.
bool wants_workspace(int64_t pairs, int64_t d, int64_t cap) {
    return d == 128 ? pairs <= 128 && cap >= 128 && cap <= 32768 : pairs <= 64 && cap >= 2048 && cap <= 32768;
}
int64_t small_parts_bytes(int64_t pairs, int64_t d, int64_t cap) {   // one partial result per 64 rows (nats.h)
    return pairs * ((cap + 63) / 64 * (d + 4) + d) * 4;
}

PyObject* status(nats_status st, const at::Tensor& out) {
    if (st != NATS_OK) return PyLong_FromLong(st);
    return THPVariable_Wrap(out);
}

// NotTaken: None; any other C++ exception as torch raises it (an allocation that fails: torch.cuda.OutOfMemoryError)
template <typename F>
PyObject* guarded(F&& f) {
    HANDLE_TH_ERRORS
    try {
        return f();
    } catch (const NotTaken&) {
        Py_RETURN_NONE;
    }
    END_HANDLE_TH_ERRORS
}

// The library's launches without the interpreter lock, as a ctypes call makes them: a launch waits where the stream's queue
// is full, and other threads go on meanwhile.
template <typename F>
nats_status unlocked(F&& f) {
    PyThreadState* const state = PyEval_SaveThread();
    const nats_status st = f();   // (a C entry: throws nothing)
    PyEval_RestoreThread(state);
    return st;
}

// The workspace of a step: the caller's, or one made for the call (kept by the tensor until the call has been enqueued) where
// memory is left for it; the step also runs without.
void set_workspace(nats_dec_params& p, PyObject* given, at::Tensor& own, const at::Tensor& like) {
    if (given != Py_None) {
        const at::Tensor& t = tensor(given);
        if (!t.is_cuda() || t.layout() != at::kStrided || !t.is_contiguous()) throw NotTaken();
        p.workspace = t.data_ptr();
        p.workspace_bytes = (size_t)t.numel();
    } else if (wants_workspace((int64_t)p.B * p.H, p.d, p.cap) && !capturing()) {
        const int64_t bytes = small_parts_bytes((int64_t)p.B * p.H, p.d, p.cap);
        try {
            own = at::empty({bytes}, like.options().dtype(at::kByte));
        } catch (const c10::OutOfMemoryError&) {
            return;
        }
        p.workspace = own.data_ptr();
        p.workspace_bytes = (size_t)bytes;
    }
}

void set_scalars(nats_dec_params& p, PyObject* const* a) {   // softmax_scale, la_scale, combine_mode, rms_eps, linear_op
    p.softmax_scale = (float)number(a[0]);
    p.la_scale = (float)number(a[1]);
    p.combine_mode = integer(a[2]);
    p.rms_eps = (float)number(a[3]);
    p.linear_op = integer(a[4]);
}

// decode(state, k_cache, v_cache, cache_len, q, k, v, alpha, beta, mask, q_nla, k_nla, w_nla, w_la, out, err_flags,
//        workspace, softmax_scale, la_scale, combine_mode, rms_eps, linear_op, freeze_on_softmax)
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        if (n != 23) throw NotTaken();
        const at::Tensor& kc = tensor(a[1]);
        if (kc.dim() != 4) throw NotTaken();
        const int64_t B = kc.size(0), H = kc.size(1), cap = kc.size(2), d = kc.size(3);
        const at::ScalarType dt = kc.scalar_type();
        nats_dec_params p{};
        p.B = (int)B; p.H = (int)H; p.d = (int)d; p.cap = (int)cap; p.dtype = dtype_code(dt);
        void* state = pointer(a[0], at::kFloat, {B, H, d, d});
        void* kcache = pointer(kc, dt, {B, H, cap, d});
        void* vcache = pointer(a[2], dt, {B, H, cap, d});
        void* len = pointer(a[3], at::kInt, {B, H});
        const at::Tensor& q = tensor(a[4]);
        void* qp = pointer(q, dt, {B, H, d});
        void* kp = pointer(a[5], dt, {B, H, d});
        void* vp = pointer(a[6], dt, {B, H, d});
        void* alpha = pointer(a[7], at::kFloat, {B, H});
        void* beta = pointer(a[8], at::kFloat, {B, H});
        void* mask = pointer(a[9], at::kByte, {B, H});
        p.q_nla = optional(a[10], dt, {B, H, d});
        p.k_nla = optional(a[11], dt, {B, H, d});
        void* wn = optional(a[12], at::kFloat, {B, H});
        void* wl = optional(a[13], at::kFloat, {B, H});
        void* err = optional(a[15], at::kInt, {B, H});
        set_scalars(p, a + 17);
        p.freeze_on_softmax = integer(a[22]);
        const at::Tensor out = a[14] == Py_None ? at::empty({B, H, d}, q.options()) : tensor(a[14]);
        void* op = pointer(out, dt, {B, H, d});
        at::Tensor own;
        set_workspace(p, a[16], own, q);
        void* const stream = current_stream();
        return status(unlocked([&] {
            return nats_hybrid_attn_decode(&p, (float*)state, kcache, vcache, (int32_t*)len, qp, kp, vp, (const float*)alpha,
                                           (const float*)beta, (const uint8_t*)mask, (const float*)wn, (const float*)wl, op,
                                           (int32_t*)err, stream);
        }), out);
    });
}

PyObject* item(PyObject* dict, const char* key) {
    PyObject* o = PyDict_GetItemString(dict, key);   // borrowed
    if (o == nullptr) throw NotTaken();
    return o;
}

// decode_chunk(st, q, k, v, alpha, beta, w_nla, w_la, out, err_flags, softmax_scale, la_scale, combine_mode, rms_eps, linear_op)
PyObject* decode_chunk(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        if (n != 15 || !PyDict_CheckExact(a[0])) throw NotTaken();
        const at::Tensor& kc = tensor(item(a[0], "k_cache"));
        if (kc.dim() != 4) throw NotTaken();
        const int64_t B = kc.size(0), H = kc.size(1), cap = kc.size(2), d = kc.size(3);
        const at::ScalarType dt = kc.scalar_type();
        nats_dec_params p{};
        p.B = (int)B; p.H = (int)H; p.d = (int)d; p.cap = (int)cap; p.dtype = dtype_code(dt);
        nats_dec_chunk_state s{};
        s.state = (float*)pointer(item(a[0], "state"), at::kFloat, {B, H, d, d});
        s.state_start = (float*)pointer(item(a[0], "state_start"), at::kFloat, {B, H, d, d});
        s.chunk_decay = (float*)pointer(item(a[0], "chunk_decay"), at::kFloat, {B, H});
        s.chunk_pos = (int32_t*)pointer(item(a[0], "chunk_pos"), at::kInt, {B, H});
        s.k_cache = pointer(kc, dt, {B, H, cap, d});
        s.v_cache = pointer(item(a[0], "v_cache"), dt, {B, H, cap, d});
        s.cache_len = (int32_t*)pointer(item(a[0], "cache_len"), at::kInt, {B, H});
        const at::Tensor& q = tensor(a[1]);
        void* qp = pointer(q, dt, {B, H, d});
        void* kp = pointer(a[2], dt, {B, H, d});
        void* vp = pointer(a[3], dt, {B, H, d});
        void* alpha = pointer(a[4], at::kFloat, {B, H});
        void* beta = pointer(a[5], at::kFloat, {B, H});
        void* wn = optional(a[6], at::kFloat, {B, H});
        void* wl = optional(a[7], at::kFloat, {B, H});
        void* err = optional(a[9], at::kInt, {B, H});
        set_scalars(p, a + 10);
        const at::Tensor out = a[8] == Py_None ? at::empty({B, H, d}, q.options()) : tensor(a[8]);
        void* op = pointer(out, dt, {B, H, d});
        at::Tensor own;
        set_workspace(p, Py_None, own, q);
        void* const stream = current_stream();
        return status(unlocked([&] {
            return nats_hybrid_attn_decode_chunk(&p, &s, qp, kp, vp, (const float*)alpha, (const float*)beta, (const float*)wn,
                                                 (const float*)wl, op, (int32_t*)err, stream);
        }), out);
    });
}

PyMethodDef methods[] = {
    {"decode", (PyCFunction)(void (*)(void))decode, METH_FASTCALL, "nats_hybrid_attn_decode"},
    {"decode_chunk", (PyCFunction)(void (*)(void))decode_chunk, METH_FASTCALL, "nats_hybrid_attn_decode_chunk"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_nats_host", "host path of the per-token calls", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__nats_host() { return PyModule_Create(&module); }
