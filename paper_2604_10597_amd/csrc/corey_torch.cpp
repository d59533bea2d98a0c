// Python extension `_native`: the calls of libcorey on torch tensors.  Marshalling only: it checks what the library
// cannot see (device, contiguity, storage types, shapes), allocates the outputs a caller left out from torch's caching
// allocator and hands pointers and the current stream to the C ABI (include/corey.h).
//
// It exists because this work was the time of every small call: from Python through ctypes a call cost 12 to 15 us of host
// time (a conversion per argument, a shape tuple per check, a stream object, a Python-level torch.empty per output) in front of
// kernels of 3 us.  Here a call costs about 2 us plus its launches.
//
// The library is found through the path binding.py loads (so COREY_LIB works): attach() takes the functions' addresses from
// that shared object.  Functions take their arguments by position; binding.py holds the signatures and defaults.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <dlfcn.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "corey.h"

namespace {

// What the library exports, as function pointers with the header's own types.
struct Lib {
#define COREY_FN(name) decltype(&::name) name
    COREY_FN(corey_entropy_hist);
    COREY_FN(corey_entropy_hist_workspace);
    COREY_FN(corey_entropy_hist_static);
    COREY_FN(corey_entropy_hist_onesweep);
    COREY_FN(corey_entropy_hist_from_table);
    COREY_FN(corey_pattern_table_workspace);
    COREY_FN(corey_policy_default);
    COREY_FN(corey_select_chunk_device);
    COREY_FN(corey_route_device);
    COREY_FN(corey_route_device_deferred);
    COREY_FN(causal_conv1d_silu_fwd);
    COREY_FN(selective_scan_fwd);
    COREY_FN(selective_scan_fwd_routed);
    COREY_FN(selective_scan_fwd_workspace);
    COREY_FN(selective_state_update);
    COREY_FN(corey_last_error);
#undef COREY_FN
};
Lib lib = {};
PyObject* error_class = nullptr;        // binding.CoreyError
PyObject* route_class = nullptr;        // binding.DeferredRoute
corey_policy default_policy;

// A Python exception is set; unwinds to the entry point, which returns NULL.
struct PyError {};

[[noreturn]] void raise(PyObject* type, const char* fmt, const char* a = "", const char* b = "")
{
    PyErr_Format(type, fmt, a, b);
    throw PyError{};
}

void check(int status)
{
    if (status == COREY_OK) return;
    PyObject* e = PyObject_CallFunction(error_class, "is", status, lib.corey_last_error());
    if (e) {
        PyErr_SetObject(error_class, e);
        Py_DECREF(e);
    }
    throw PyError{};
}

// ------------------------------------------------------------------------------------------- arguments
// A tensor argument; NULL for None.  The reference stays the caller's.
const at::Tensor* optional_tensor(PyObject* o, const char* name)
{
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) raise(PyExc_TypeError, "%s must be a tensor", name);
    const at::Tensor* t = &THPVariable_Unpack(o);
    if (!t->is_cuda() || !t->is_contiguous()) raise(PyExc_ValueError, "%s must be a contiguous GPU tensor", name);
    return t;
}

const at::Tensor& tensor(PyObject* o, const char* name)
{
    const at::Tensor* t = optional_tensor(o, name);
    if (!t) raise(PyExc_TypeError, "%s must be a tensor", name);
    return *t;
}

// The (optional) tensor must have this type and shape: the library reads raw memory and cannot check either.
void want(const at::Tensor* t, const char* name, at::ScalarType type, at::IntArrayRef shape)
{
    if (!t || (t->scalar_type() == type && t->sizes() == shape)) return;
    std::string s = c10::toString(type);
    s += " of shape (";
    for (size_t i = 0; i < shape.size(); ++i) s += (i ? ", " : "") + std::to_string(shape[i]);
    raise(PyExc_TypeError, "%s must be %s)", name, s.c_str());
}

void want(const at::Tensor& t, const char* name, at::ScalarType type, at::IntArrayRef shape)
{
    if (t.defined()) want(&t, name, type, shape);
}

// Memory kernels reach: on the GPU, or host memory pinned for it (results may go straight there).
void want_reachable(const at::Tensor& t, const char* name)
{
    if (!(t.is_cuda() || t.is_pinned()) || !t.is_contiguous()) raise(PyExc_ValueError, "%s must be a contiguous GPU tensor", name);
}

// A tensor argument the kernels read or write through its pointer: of this type and with room for n values.  Its shape is the
// caller's business (counts of one histogram may be [K], an output longer than needed is filled at its start).
void want_room(const at::Tensor* t, const char* name, at::ScalarType type, int64_t n)
{
    if (!t) return;
    const at::ScalarType have = t->scalar_type();
    if ((have == type || (type == at::kInt && have == at::kUInt32)) && t->numel() >= n) return;      // (counts and chunks: 32-bit patterns either way)
    const std::string s = std::string(c10::toString(type)) + " with room for " + std::to_string(n) + " values";
    raise(PyExc_TypeError, "%s must be %s", name, s.c_str());
}
// ... an entry of a result dict, which nobody has looked at yet
void want_room(const at::Tensor& t, const char* name, at::ScalarType type, int64_t n)
{
    if (!t.defined()) return;
    want_reachable(t, name);
    want_room(&t, name, type, n);
}
// ... of at least n bytes, whatever its type (workspaces)
void want_bytes(const at::Tensor* t, const char* name, int64_t n)
{
    if (!t || !t->defined()) return;
    want_reachable(*t, name);
    if ((int64_t)t->nbytes() >= n) return;
    raise(PyExc_TypeError, "%s must have at least %s bytes", name, std::to_string(n).c_str());
}

corey_dtype dtype_code(at::ScalarType t)
{
    if (t == at::kFloat) return COREY_F32;
    if (t == at::kBFloat16) return COREY_BF16;
    if (t == at::kHalf) return COREY_F16;
    raise(PyExc_TypeError, "unsupported storage type %s", c10::toString(t));
}

// A whole number: an int or what offers itself as one (__index__); floats and strings are refused, not truncated or parsed.
int64_t integer(PyObject* o)
{
    PyObject* n = PyNumber_Index(o);
    if (!n) throw PyError{};
    const int64_t v = PyLong_AsLongLong(n);
    Py_DECREF(n);
    if (v == -1 && PyErr_Occurred()) throw PyError{};
    return v;
}

// What int(o) and float(o) make of it, for the arguments that are converted so: `chunk`, L of the chunk rule, `ema_lambda`.
struct Converted {
    PyObject* o;
    explicit Converted(PyObject* p) : o(p)
    {
        if (!o) throw PyError{};
    }
    ~Converted() { Py_DECREF(o); }
    Converted(const Converted&) = delete;
};

int32_t integer32(PyObject* o)
{
    const int64_t v = integer(o);
    if (v != (int32_t)v) raise(PyExc_OverflowError, "integer does not fit 32 bits");
    return (int32_t)v;
}

double number(PyObject* o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw PyError{};
    return v;
}

bool truth(PyObject* o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw PyError{};
    return v != 0;
}

// The memory of a ctypes structure (Policy, DeferredRoute).
template <typename S> S* structure(PyObject* o, const char* name)
{
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_WRITABLE) != 0) throw PyError{};
    void* p = b.buf;
    const bool fits = (size_t)b.len == sizeof(S);
    PyBuffer_Release(&b);                           // a ctypes structure keeps its memory for as long as it lives
    if (!fits) raise(PyExc_TypeError, "%s has the wrong size", name);
    return static_cast<S*>(p);
}

const corey_policy* policy_or_default(PyObject* o) { return o == Py_None ? &default_policy : structure<corey_policy>(o, "policy"); }

void* ptr(const at::Tensor* t) { return t ? t->data_ptr() : nullptr; }
void* ptr(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }
template <typename P> P* ptr_as(const at::Tensor* t) { return static_cast<P*>(ptr(t)); }
template <typename P> P* ptr_as(const at::Tensor& t) { return static_cast<P*>(ptr(t)); }

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

at::Tensor empty(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like)
{
    return at::detail::empty_cuda(shape, type, like.device(), std::nullopt);
}

PyObject* wrap(const at::Tensor& t)
{
    PyObject* o = THPVariable_Wrap(t);
    if (!o) throw PyError{};
    return o;
}

// The library only enqueues kernels, but a full queue makes the runtime wait: other threads may run meanwhile.
template <typename F> void call(F&& f)
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    check(status);
}

struct Shape3 {
    int64_t B, D, L;
};
Shape3 shape3(const at::Tensor& x)
{
    if (x.dim() != 3) raise(PyExc_ValueError, "x must be [B, D, L]");
    return {x.size(0), x.size(1), x.size(2)};
}

// ------------------------------------------------------------------------------------------- the result dict
struct Owned {                          // a reference that goes with its scope
    PyObject* o;
    explicit Owned(PyObject* p) : o(p) {}
    ~Owned() { Py_XDECREF(o); }
    PyObject* release()
    {
        PyObject* p = o;
        o = nullptr;
        return p;
    }
    Owned(const Owned&) = delete;
};

// A new reference to out[key]; for an `optional` one out.get(key) or NULL.  `out` is any mapping, in practice a dict.
PyObject* out_entry(PyObject* out, const char* key, bool optional)
{
    PyObject* o;
    if (PyDict_CheckExact(out)) {
        o = PyDict_GetItemString(out, key);
        if (!o && !optional) raise(PyExc_KeyError, "%s", key);
        Py_XINCREF(o);
        return o;
    }
    o = optional ? PyObject_CallMethod(out, "get", "s", key) : PyMapping_GetItemString(out, key);
    if (!o) throw PyError{};
    return o;
}

// out[key], which must be there (KeyError otherwise) unless `optional`; undefined for None.  The tensor is held, not borrowed:
// other Python code (another thread, once the library is called without the interpreter lock; an argument's __float__) may take
// it out of the dict before the work on it is enqueued, and its memory must not go to another tensor by then.
at::Tensor out_tensor(PyObject* out, const char* key, bool optional = false)
{
    const Owned e(out_entry(out, key, optional));
    if (!e.o || e.o == Py_None) return at::Tensor();
    if (!THPVariable_Check(e.o)) raise(PyExc_TypeError, "out[%s] must be a tensor", key);
    return THPVariable_Unpack(e.o);
}

void put(PyObject* out, const char* key, PyObject* o)
{
    if (PyDict_CheckExact(out) ? PyDict_SetItemString(out, key, o) : PyMapping_SetItemString(out, key, o)) throw PyError{};
}

void put(PyObject* out, const char* key, const at::Tensor& t) { put(out, key, Owned(wrap(t)).o); }

// A new reference to the dict to fill: the caller's, or a new one with new tensors.
PyObject* result_dict(PyObject* out, int64_t nh, int64_t K, bool with_chunks, const at::Tensor& like)
{
    if (out != Py_None) {
        Py_INCREF(out);
        return out;
    }
    PyObject* d = PyDict_New();
    if (!d) throw PyError{};
    try {
        put(d, "counts", empty({nh, K}, at::kInt, like));          // uint32 bit patterns
        put(d, "H", empty({nh}, at::kDouble, like));
        put(d, "r", empty({nh}, at::kDouble, like));
        put(d, "range", empty({nh, 2}, at::kFloat, like));
        if (with_chunks) put(d, "chunks", empty({nh}, at::kInt, like));
    } catch (...) {
        Py_DECREF(d);
        throw;
    }
    return d;
}

// The tensors of the result dict.
struct Results {
    at::Tensor counts, H, r, range;
    Results(PyObject* out, int64_t nh, int64_t K)
        : counts(out_tensor(out, "counts")), H(out_tensor(out, "H")), r(out_tensor(out, "r")), range(out_tensor(out, "range", true))
    {
        want_room(counts, "counts", at::kInt, K > 0 ? nh * K : 0);      // (the library refuses any other K)
        want_room(H, "H", at::kDouble, nh);
        want_room(r, "r", at::kDouble, nh);
        want_room(range, "range", at::kFloat, 2 * nh);
    }
};

// The workspace tensor of a statistic: the argument, the dict's, or a new one.
at::Tensor statistic_workspace(PyObject* arg, PyObject* out, bool from_dict, int64_t B, int32_t K, const at::Tensor& x)
{
    at::Tensor given;
    if (arg != Py_None) {
        if (!THPVariable_Check(arg)) raise(PyExc_TypeError, "workspace must be a tensor");
        given = THPVariable_Unpack(arg);
    } else if (from_dict) {
        given = out_tensor(out, "workspace", true);
    }
    want_bytes(&given, "workspace", 0);                         // (the library checks how many)
    if (given.defined()) return given;
    const int64_t need = (int64_t)lib.corey_entropy_hist_workspace(B, K);
    return empty({need < 256 ? 256 : need}, at::kByte, x);
}

// ------------------------------------------------------------------------------------------- entry points
// Python-visible functions take exactly N positional arguments.
template <PyObject* (*F)(PyObject* const*), int N>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
        return nullptr;
    }
    if (!error_class) {
        PyErr_SetString(PyExc_RuntimeError, "libcorey is not attached");
        return nullptr;
    }
    HANDLE_TH_ERRORS                    // torch's own errors (out of memory, ...) as the exceptions torch raises
    try {
        return F(a);
    } catch (const PyError&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

PyObject* state_update(PyObject* const* a)
{
    const at::Tensor& state = tensor(a[0], "state");
    const at::Tensor& x = tensor(a[1], "x");
    const at::Tensor& delta = tensor(a[2], "delta");
    const at::Tensor& A = tensor(a[3], "A");
    const at::Tensor& Bt = tensor(a[4], "Bt");
    const at::Tensor& Ct = tensor(a[5], "Ct");
    const at::Tensor* Dv = optional_tensor(a[6], "Dv");
    const at::Tensor* z = optional_tensor(a[7], "z");
    const at::Tensor* bias = optional_tensor(a[8], "delta_bias");
    const int softplus = truth(a[9]) ? 1 : 0;
    const at::Tensor* y = optional_tensor(a[10], "y");
    if (state.dim() != 3) raise(PyExc_ValueError, "state must be [B, D, N]");
    const int64_t B = state.size(0), D = state.size(1), N = state.size(2);
    const at::ScalarType type = x.scalar_type();
    if (state.scalar_type() != at::kFloat || A.scalar_type() != at::kFloat || A.sizes() != at::IntArrayRef({D, N}))
        raise(PyExc_TypeError, "state [B, D, N] and A [D, N] must be float32");
    want(&x, "x", type, {B, D});
    want(&delta, "delta", type, {B, D});
    want(z, "z", type, {B, D});
    want(&Bt, "Bt", type, {B, N});
    want(&Ct, "Ct", type, {B, N});
    want(Dv, "Dv", at::kFloat, {D});
    want(bias, "delta_bias", at::kFloat, {D});
    want_room(y, "y", type, B * D);
    const corey_dtype dt = dtype_code(type);
    at::Tensor made;
    if (!y) {
        made = empty({B, D}, type, x);
        y = &made;
    }
    void* s = stream();
    call([&] {
        return lib.selective_state_update(ptr(state), ptr(x), ptr(delta), ptr_as<float>(A), ptr(Bt), ptr(Ct), ptr_as<float>(Dv), ptr(z),
                                          ptr_as<float>(bias), softplus, ptr(y), dt, B, D, N, s);
    });
    if (y != &made) {
        Py_INCREF(a[10]);
        return a[10];
    }
    return wrap(made);
}

PyObject* conv(PyObject* const* a)
{
    const at::Tensor& x = tensor(a[0], "x");
    const at::Tensor& weight = tensor(a[1], "weight");
    const at::Tensor* bias = optional_tensor(a[2], "bias");
    const at::Tensor* state_in = optional_tensor(a[3], "state_in");
    const at::Tensor* u = optional_tensor(a[4], "u");
    const bool want_state = truth(a[5]);
    const at::Tensor* parts = optional_tensor(a[6], "range_parts");
    const at::Tensor* table = optional_tensor(a[7], "pattern_table");
    const Shape3 g = shape3(x);
    if (weight.dim() != 2 || weight.size(0) != g.D || weight.scalar_type() != at::kFloat || (bias && bias->scalar_type() != at::kFloat))
        raise(PyExc_TypeError, "weight [D, W] and bias [D] must be float32");
    const int64_t W = weight.size(1);
    const corey_dtype dt = dtype_code(x.scalar_type());
    want_room(bias, "bias", at::kFloat, g.D);
    want_room(state_in, "state_in", x.scalar_type(), g.B * g.D * (W - 1));
    want_room(u, "u", x.scalar_type(), g.B * g.D * g.L);
    at::Tensor made_u, made_state, made_parts;
    if (!u) {
        made_u = empty({g.B, g.D, g.L}, x.scalar_type(), x);
        u = &made_u;
    }
    if (want_state) made_state = empty({g.B, g.D, W - 1}, x.scalar_type(), x);
    if (!parts) {
        made_parts = empty({COREY_HANDOFF_BYTES}, at::kByte, x);
        parts = &made_parts;
    } else if (parts->numel() < COREY_HANDOFF_BYTES || parts->scalar_type() != at::kByte) {
        raise(PyExc_TypeError, "range_parts must be a uint8 tensor of %s bytes", std::to_string(COREY_HANDOFF_BYTES).c_str());
    }
    void* s = stream();
    call([&] {
        return lib.causal_conv1d_silu_fwd(ptr(x), ptr_as<float>(weight), ptr_as<float>(bias), ptr(state_in), ptr(u),
                                          want_state ? made_state.data_ptr() : nullptr, ptr(parts), ptr(table),
                                          table ? (size_t)table->numel() : 0, dt, g.B, g.D, g.L, (int32_t)W, s);
    });
    Owned ru(u == &made_u ? wrap(made_u) : (Py_INCREF(a[4]), a[4]));
    Owned rs(want_state ? wrap(made_state) : (Py_INCREF(Py_None), Py_None));
    Owned rp(parts == &made_parts ? wrap(made_parts) : (Py_INCREF(a[6]), a[6]));
    return PyTuple_Pack(3, ru.o, rs.o, rp.o);
}

PyObject* hist(PyObject* const* a)      // x, K, eps, stride, seqlens, out, workspace, block, range_parts
{
    const at::Tensor& x = tensor(a[0], "x");
    const at::Tensor* seqlens = optional_tensor(a[4], "seqlens");
    const Shape3 g = shape3(x);
    const int64_t nh = seqlens ? g.B : 1;
    want(seqlens, "seqlens", at::kInt, {g.B});
    const int32_t K = integer32(a[1]);
    const double eps = number(a[2]);
    const int64_t stride = integer(a[3]), block = integer(a[7]);
    const at::Tensor* parts = optional_tensor(a[8], "range_parts");
    want_bytes(parts, "range_parts", COREY_HANDOFF_BYTES);
    const corey_dtype dt = dtype_code(x.scalar_type());
    Owned out(result_dict(a[5], nh, K, false, x));
    const at::Tensor ws = statistic_workspace(a[6], out.o, false, g.B, K, x);
    const Results o(out.o, nh, K);
    void* s = stream();
    call([&] {
        return lib.corey_entropy_hist(ptr(x), dt, g.B, g.D, g.L, ptr_as<int32_t>(seqlens), K, eps, stride, block, ptr_as<uint32_t>(o.counts),
                                      ptr_as<double>(o.H), ptr_as<double>(o.r), ptr_as<float>(o.range), ptr(parts), ptr(ws),
                                      (size_t)ws.numel(), s);
    });
    put(out.o, "workspace", ws);
    return out.release();
}

PyObject* hist_static(PyObject* const* a)      // x, K, out, eps, stride, seqlens, block, range_parts
{
    const at::Tensor& x = tensor(a[0], "x");
    const at::Tensor* seqlens = optional_tensor(a[5], "seqlens");
    const Shape3 g = shape3(x);
    const int64_t nh = seqlens ? g.B : 1;
    want(seqlens, "seqlens", at::kInt, {g.B});
    const int32_t K = integer32(a[1]);
    const Results o(a[2], nh, K);
    want(o.counts, "counts", at::kInt, {nh, K});
    want(o.H, "H", at::kDouble, {nh});
    want(o.r, "r", at::kDouble, {nh});
    want(o.range, "range", at::kFloat, {nh, 2});
    const double eps = number(a[3]);
    const int64_t stride = integer(a[4]), block = integer(a[6]);
    const at::Tensor* parts = optional_tensor(a[7], "range_parts");
    want_bytes(parts, "range_parts", COREY_HANDOFF_BYTES);
    const corey_dtype dt = dtype_code(x.scalar_type());
    void* s = stream();
    call([&] {
        return lib.corey_entropy_hist_static(ptr(x), dt, g.B, g.D, g.L, ptr_as<int32_t>(seqlens), K, eps, stride, block,
                                             ptr_as<uint32_t>(o.counts), ptr_as<double>(o.H), ptr_as<double>(o.r), ptr_as<float>(o.range),
                                             ptr(parts), s);
    });
    Py_INCREF(a[2]);
    return a[2];
}

// Both forms of the one-sweep statistic: the arguments after the tensor or table.
struct TableCall {
    const corey_policy* policy = nullptr;
    at::Tensor chunks;
    Results o;
    TableCall(PyObject* p, PyObject* out, int64_t K, const at::Tensor& like) : o(out, 1, K)
    {
        if (p == Py_None) return;
        policy = structure<corey_policy>(p, "policy");
        chunks = out_tensor(out, "chunks", true);
        want_room(chunks, "chunks", at::kInt, 1);
        if (chunks.defined()) return;
        chunks = empty({1}, at::kInt, like);
        put(out, "chunks", chunks);
    }
};

PyObject* onesweep(PyObject* const* a)      // x, K, eps, policy, out, table_ws
{
    const at::Tensor& x = tensor(a[0], "x");
    const at::Tensor* ws = optional_tensor(a[5], "table_ws");
    const Shape3 g = shape3(x);
    const int32_t K = integer32(a[1]);
    const double eps = number(a[2]);
    const corey_dtype dt = dtype_code(x.scalar_type());
    Owned out(result_dict(a[4], 1, K, false, x));
    const TableCall t(a[3], out.o, K, x);
    at::Tensor made;
    if (!ws) {
        made = empty({(int64_t)lib.corey_pattern_table_workspace()}, at::kByte, x);
        ws = &made;
    }
    void* s = stream();
    call([&] {
        return lib.corey_entropy_hist_onesweep(ptr(x), dt, g.B, g.D, g.L, K, eps, t.policy, ptr_as<int32_t>(t.chunks),
                                               ptr_as<uint32_t>(t.o.counts), ptr_as<double>(t.o.H), ptr_as<double>(t.o.r),
                                               ptr_as<float>(t.o.range), ptr(ws), (size_t)ws->numel(), s);
    });
    put(out.o, "table_ws", *ws);
    return out.release();
}

PyObject* from_table(PyObject* const* a)      // table_ws, dtype code, L, K, eps, policy, out
{
    const at::Tensor& ws = tensor(a[0], "table_ws");
    const corey_dtype dt = (corey_dtype)integer32(a[1]);
    const int64_t L = integer(a[2]);
    const int32_t K = integer32(a[3]);
    const double eps = number(a[4]);
    Owned out(result_dict(a[6], 1, K, false, ws));
    const TableCall t(a[5], out.o, K, ws);
    void* s = stream();
    call([&] {
        return lib.corey_entropy_hist_from_table(dt, L, K, eps, t.policy, ptr_as<int32_t>(t.chunks), ptr_as<uint32_t>(t.o.counts),
                                                 ptr_as<double>(t.o.H), ptr_as<double>(t.o.r), ptr_as<float>(t.o.range), ptr(ws),
                                                 (size_t)ws.numel(), s);
    });
    return out.release();
}

// corey_route_device and its deferred form: x, K, policy, eps, stride, block, seqlens, out, workspace, chunk_calls,
// range_parts, then ema_lambda and ema_state where there is a reduction of its own.
template <bool DEFERRED> PyObject* route(PyObject* const* a)
{
    const at::Tensor* calls = optional_tensor(a[9], "chunk_calls");
    const at::Tensor& x = tensor(a[0], "x");
    const at::Tensor* seqlens = optional_tensor(a[6], "seqlens");
    const Shape3 g = shape3(x);
    const int64_t nh = seqlens ? g.B : 1;
    want(seqlens, "seqlens", at::kInt, {g.B});
    want(calls, "chunk_calls", at::kInt, {COREY_CHUNK_SLOTS});
    const int32_t K = integer32(a[1]);
    const corey_policy* p = policy_or_default(a[2]);
    const double eps = number(a[3]);
    const int64_t stride = integer(a[4]), block = integer(a[5]);
    const at::Tensor* parts = optional_tensor(a[10], "range_parts");
    want_bytes(parts, "range_parts", COREY_HANDOFF_BYTES);
    const corey_dtype dt = dtype_code(x.scalar_type());
    Owned out(result_dict(a[7], nh, K, true, x));
    const at::Tensor ws = statistic_workspace(a[8], out.o, true, g.B, K, x);
    const Results o(out.o, nh, K);
    const at::Tensor chunks = out_tensor(out.o, "chunks");
    want_room(chunks, "chunks", at::kInt, nh);
    const int32_t* lens = ptr_as<int32_t>(seqlens);
    uint32_t* cc = ptr_as<uint32_t>(calls);
    void* s = stream();
    if constexpr (DEFERRED) {
        const Owned given(out_entry(out.o, "route", true));
        const Owned ticket(given.o && given.o != Py_None ? (Py_INCREF(given.o), given.o) : PyObject_CallNoArgs(route_class));
        if (!ticket.o) throw PyError{};
        corey_deferred_route* t = structure<corey_deferred_route>(ticket.o, "route");
        call([&] {
            return lib.corey_route_device_deferred(ptr(x), dt, g.B, g.D, g.L, lens, K, eps, stride, block, p, cc, ptr_as<uint32_t>(o.counts),
                                                   ptr_as<double>(o.H), ptr_as<double>(o.r), ptr_as<float>(o.range), ptr(parts),
                                                   ptr_as<int32_t>(chunks), ptr(ws), (size_t)ws.numel(), t, s);
        });
        put(out.o, "workspace", ws);
        put(out.o, "route", ticket.o);
    } else {
        const double lambda = number(Converted(PyNumber_Float(a[11])).o);
        const at::Tensor* ema = optional_tensor(a[12], "ema_state");
        want(ema, "ema_state", at::kDouble, {nh});
        call([&] {
            return lib.corey_route_device(ptr(x), dt, g.B, g.D, g.L, lens, K, eps, stride, block, p, lambda, ptr_as<double>(ema), cc,
                                          ptr_as<uint32_t>(o.counts), ptr_as<double>(o.H), ptr_as<double>(o.r), ptr_as<float>(o.range),
                                          ptr(parts), ptr_as<int32_t>(chunks), ptr(ws), (size_t)ws.numel(), s);
        });
        put(out.o, "workspace", ws);
    }
    return out.release();
}

PyObject* select_chunk_device(PyObject* const* a)      // r_dev, L, policy, seqlens, out
{
    const at::Tensor& r = tensor(a[0], "r_dev");
    const at::Tensor* seqlens = optional_tensor(a[3], "seqlens");
    if (r.scalar_type() != at::kDouble) raise(PyExc_TypeError, "r_dev must be float64");
    const int64_t nh = r.numel();
    want(seqlens, "seqlens", at::kInt, {nh});
    const corey_policy* p = policy_or_default(a[2]);
    const int64_t L = integer(Converted(PyNumber_Long(a[1])).o);
    at::Tensor made;
    const at::Tensor* out = optional_tensor(a[4], "out");
    want_room(out, "out", at::kInt, nh);
    if (!out) {
        made = empty({nh}, at::kInt, r);
        out = &made;
    }
    void* s = stream();
    call([&] { return lib.corey_select_chunk_device(ptr_as<double>(r), ptr_as<int32_t>(seqlens), L, (int32_t)nh, p, ptr_as<int32_t>(out), s); });
    if (out != &made) {
        Py_INCREF(a[4]);
        return a[4];
    }
    return wrap(made);
}

PyObject* scan(PyObject* const* a)
{
    const at::Tensor& u = tensor(a[0], "u");
    const at::Tensor& delta = tensor(a[1], "delta");
    const at::Tensor& A = tensor(a[2], "A");
    const at::Tensor& Bm = tensor(a[3], "Bm");
    const at::Tensor& Cm = tensor(a[4], "Cm");
    const at::Tensor* Dv = optional_tensor(a[5], "Dv");
    const at::Tensor* z = optional_tensor(a[6], "z");
    const at::Tensor* bias = optional_tensor(a[7], "delta_bias");
    const int softplus = truth(a[8]) ? 1 : 0;
    const at::Tensor* h0 = optional_tensor(a[9], "h0");
    const at::Tensor* seqlens = optional_tensor(a[10], "seqlens");
    const int32_t chunk = integer32(Converted(PyNumber_Long(a[11])).o);
    const at::Tensor* chunks = optional_tensor(a[12], "chunks_dev");
    const at::Tensor* y = optional_tensor(a[13], "y");
    const at::Tensor* last = optional_tensor(a[14], "last_state");
    const at::Tensor* ws = optional_tensor(a[15], "workspace");
    uint32_t flags = (truth(a[16]) ? COREY_SCAN_GENERAL_A : 0u) | (truth(a[18]) ? COREY_SCAN_WHOLE_ROWS : 0u);
    if (u.dim() != 3 || A.dim() != 2) raise(PyExc_ValueError, "u must be [B, D, L] and A [D, N]");
    const int64_t B = u.size(0), D = u.size(1), L = u.size(2), N = A.size(1);
    const int64_t bnl[3] = {B, N, L};
    if (A.size(0) != D || Bm.sizes() != at::IntArrayRef(bnl) || Cm.sizes() != at::IntArrayRef(bnl) || delta.sizes() != u.sizes()) raise(PyExc_ValueError, "inconsistent shapes");
    const at::ScalarType type = u.scalar_type();
    want(&delta, "delta", type, {B, D, L});
    want(z, "z", type, {B, D, L});
    want(y, "y", type, {B, D, L});
    want(&Bm, "Bm", type, {B, N, L});
    want(&Cm, "Cm", type, {B, N, L});
    want(&A, "A", at::kFloat, {D, N});
    want(Dv, "Dv", at::kFloat, {D});
    want(bias, "delta_bias", at::kFloat, {D});
    want(h0, "h0", at::kFloat, {B, D, N});
    want(last, "last_state", at::kFloat, {B, D, N});
    want(seqlens, "seqlens", at::kInt, {B});
    // a single routed chunk (the whole-tensor statistic of a batch) applies to every sequence
    const bool one_chunk = chunks && B > 1 && chunks->dim() == 1 && chunks->size(0) == 1;
    want(chunks, "chunks_dev", at::kInt, {one_chunk ? 1 : B});
    const corey_dtype dt = dtype_code(type);
    if (a[17] != Py_None && chunks) raise(PyExc_ValueError, "a route brings its own chunks");
    const corey_deferred_route* ticket = a[17] != Py_None ? structure<corey_deferred_route>(a[17], "route") : nullptr;
    at::Tensor made_y, made_last, made_ws;
    if (!y) {
        made_y = empty({B, D, L}, type, u);
        y = &made_y;
    }
    if (!last) {
        made_last = empty({B, D, N}, at::kFloat, u);
        last = &made_last;
    }
    if (!ws) {
        made_ws = empty({(int64_t)lib.selective_scan_fwd_workspace(B, N, L)}, at::kByte, u);
        ws = &made_ws;
    }
    void* s = stream();
    const size_t ws_bytes = (size_t)ws->numel();
    if (ticket)
        call([&] {
            return lib.selective_scan_fwd_routed(ptr(u), ptr(delta), ptr_as<float>(A), ptr(Bm), ptr(Cm), ptr_as<float>(Dv), ptr(z),
                                                 ptr_as<float>(bias), softplus, ptr_as<float>(h0), ptr_as<int32_t>(seqlens), chunk, ticket,
                                                 ptr(y), ptr_as<float>(last), dt, B, D, N, L, flags, ptr(ws), ws_bytes, s);
        });
    else
        call([&] {
            return lib.selective_scan_fwd(ptr(u), ptr(delta), ptr_as<float>(A), ptr(Bm), ptr(Cm), ptr_as<float>(Dv), ptr(z),
                                          ptr_as<float>(bias), softplus, ptr_as<float>(h0), ptr_as<int32_t>(seqlens), chunk,
                                          ptr_as<int32_t>(chunks), ptr(y), ptr_as<float>(last), dt, B, D, N, L,
                                          flags | (one_chunk ? COREY_SCAN_ONE_CHUNK : 0u), ptr(ws), ws_bytes, s);
        });
    Owned ry(y == &made_y ? wrap(made_y) : (Py_INCREF(a[13]), a[13]));
    Owned rl(last == &made_last ? wrap(made_last) : (Py_INCREF(a[14]), a[14]));
    return PyTuple_Pack(2, ry.o, rl.o);
}

// attach(path of libcorey.so, CoreyError, DeferredRoute): take the library's functions.  The library is loaded already.
PyObject* attach(PyObject*, PyObject* args)
{
    const char* path;
    PyObject *err, *rt;
    if (!PyArg_ParseTuple(args, "sOO", &path, &err, &rt)) return nullptr;
    void* h = dlopen(path, RTLD_NOW);
    if (!h) {
        PyErr_SetString(PyExc_ImportError, dlerror());
        return nullptr;
    }
    Lib l = {};
#define COREY_FN(name)                                                                      \
    l.name = reinterpret_cast<decltype(l.name)>(dlsym(h, #name));                           \
    if (!l.name) {                                                                          \
        PyErr_SetString(PyExc_ImportError, "libcorey lacks " #name);                        \
        return nullptr;                                                                     \
    }
    COREY_FN(corey_entropy_hist)
    COREY_FN(corey_entropy_hist_workspace)
    COREY_FN(corey_entropy_hist_static)
    COREY_FN(corey_entropy_hist_onesweep)
    COREY_FN(corey_entropy_hist_from_table)
    COREY_FN(corey_pattern_table_workspace)
    COREY_FN(corey_policy_default)
    COREY_FN(corey_select_chunk_device)
    COREY_FN(corey_route_device)
    COREY_FN(corey_route_device_deferred)
    COREY_FN(causal_conv1d_silu_fwd)
    COREY_FN(selective_scan_fwd)
    COREY_FN(selective_scan_fwd_routed)
    COREY_FN(selective_scan_fwd_workspace)
    COREY_FN(selective_state_update)
    COREY_FN(corey_last_error)
#undef COREY_FN
    lib = l;
    if (lib.corey_policy_default(&default_policy) != COREY_OK) {
        PyErr_SetString(PyExc_ImportError, "libcorey gave no default policy");
        return nullptr;
    }
    Py_INCREF(rt);
    Py_XSETREF(route_class, rt);
    Py_INCREF(err);
    Py_XSETREF(error_class, err);
    Py_RETURN_NONE;
}

#define COREY_ENTRY(name, f, n) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<f, n>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"attach", attach, METH_VARARGS, nullptr},
    COREY_ENTRY("selective_state_update", state_update, 11),
    COREY_ENTRY("causal_conv1d_silu_fwd", conv, 8),
    COREY_ENTRY("corey_entropy_hist", hist, 9),
    COREY_ENTRY("corey_entropy_hist_static", hist_static, 8),
    COREY_ENTRY("corey_entropy_hist_onesweep", onesweep, 6),
    COREY_ENTRY("corey_entropy_hist_from_table", from_table, 7),
    COREY_ENTRY("corey_route_device", route<false>, 13),
    COREY_ENTRY("corey_route_device_deferred", route<true>, 11),
    COREY_ENTRY("corey_select_chunk_device", select_chunk_device, 5),
    COREY_ENTRY("selective_scan_fwd", scan, 19),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "libcorey on torch tensors", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
