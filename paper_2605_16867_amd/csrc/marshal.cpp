// Argument marshalling of the calls of a serving loop, in native code: a call of a dozen tensors spends 7 to 9 us
// in the interpreter when each of them is checked there (type, place, layout, size, address), several times what
// the call itself takes to queue its kernels; here it is below one.  What is accepted and what is refused is the same: an
// argument that is not plainly right (a subclass, a wrong type, too short) goes to the binding's own check,
// which raises, or knows it to be right after all.
//
// No kernel and no routing arithmetic here, and no link to the library: the binding hands over the addresses
// of the entry points it has loaded (connect).
#include <Python.h>

#include <ATen/core/TensorBase.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>

namespace {

using std::int32_t;
using std::int64_t;

struct Entries {
    int (*build_status)(void*, const void*, const void*, const void*, const void*, int64_t, const void*, const void*,
                        const void*, int64_t, void*, void*, void*, void*, void*);
    int (*score_route)(void*, int64_t, const void*, const void*, const void*, const void*, void*, void*, void*, void*, void*);
    int (*score_route_noalloc)(void*, int64_t, const void*, const void*, const void*, const void*, void*, void*, void*, void*);
    int (*score_route_cached)(void*, int64_t, const void*, const void*, const void*, const void*, const void*, const void*,
                              const void*, int64_t, void*, void*, void*, void*, void*);
    int (*route_feedback)(void*, int64_t, int64_t, const void*, const void*, const void*, const void*, void*, void*, void*, void*);
    int (*risk_scan)(void*, const void*, const void*, const void*, const void*, int64_t, const void*, const void*, const void*,
                     int64_t, const void*, void*, void*, void*, void*, void*, void*);
} entries;

PyObject* check_slowly = nullptr;      // (tensor, type code, name, elements or None) -> address or None, or raises

struct Raised {};      // a Python exception is set

constexpr int64_t kAny = -1;

int64_t numel(PyObject* o)
{
    if (THPVariable_CheckExact(o)) return THPVariable_Unpack(o).numel();
    PyObject* n = PyObject_CallMethod(o, "numel", nullptr);
    if (!n) throw Raised{};
    const long long v = PyLong_AsLongLong(n);
    Py_DECREF(n);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
}

// The address of a contiguous GPU tensor of the type with at least `need` elements; None: null.
void* address(PyObject* o, at::ScalarType type, const char* name, int64_t need = kAny)
{
    if (o == Py_None) return nullptr;
    if (THPVariable_CheckExact(o)) {
        const at::TensorBase& t = THPVariable_Unpack(o);
        if (t.is_cuda() && t.scalar_type() == type && t.is_contiguous() && t.numel() >= need) return t.data_ptr();
    }
    const char* code = type == at::kInt ? "i" : type == at::kFloat ? "f" : type == at::kDouble ? "d" : "B";
    PyObject* r = need == kAny ? PyObject_CallFunction(check_slowly, "OssO", o, code, name, Py_None)
                               : PyObject_CallFunction(check_slowly, "OssL", o, code, name, (long long)need);
    if (!r) throw Raised{};
    void* p = r == Py_None ? nullptr : PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    if (PyErr_Occurred()) throw Raised{};
    return p;
}

void* i32(PyObject* o, const char* name, int64_t need = kAny) { return address(o, at::kInt, name, need); }
void* f32(PyObject* o, const char* name, int64_t need = kAny) { return address(o, at::kFloat, name, need); }
void* f64(PyObject* o, const char* name, int64_t need = kAny) { return address(o, at::kDouble, name, need); }
void* u8(PyObject* o, const char* name, int64_t need = kAny) { return address(o, at::kByte, name, need); }

void* handle(PyObject* o)
{
    if (o == Py_None) return nullptr;
    void* p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw Raised{};
    return p;
}

int64_t integer(PyObject* o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
}

// torch's current stream on its current device
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// (the library's calls do not touch Python objects: other threads may run meanwhile)
template <typename... P, typename... A>
PyObject* call(int (*entry)(P...), A... args)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = entry(args...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

template <Py_ssize_t kArgs, PyObject* (*kCall)(PyObject* const*)>
PyObject* guarded(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != kArgs) { PyErr_Format(PyExc_TypeError, "need %zd arguments, got %zd", kArgs, n); return nullptr; }
    try {
        return kCall(a);
    } catch (const Raised&) {
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

// Arguments of each: the handle's address, then what the comment says, in the order of the binding's methods.

// n_inst, act_off, act_prompt, act_gen, act_rem, q_off, q_prompt, q_len, out_act_finish, out_q_finish, out_d, out_rank
PyObject* build_status(PyObject* const* a)
{
    const int64_t M = integer(a[1]), na = numel(a[3]), nq = numel(a[7]);
    void* const act_off = i32(a[2], "act_off", M + 1);
    void* const act_prompt = i32(a[3], "act_prompt");
    void* const act_gen = i32(a[4], "act_gen", na);
    void* const act_rem = i32(a[5], "act_rem", na);
    void* const q_off = i32(a[6], "q_off", M + 1);
    void* const q_prompt = i32(a[7], "q_prompt");
    void* const q_len = i32(a[8], "q_len", nq);
    void* const finish = f32(a[9], "out_act_finish", na);
    void* const q_finish = f32(a[10], "out_q_finish", nq);
    void* const d = f64(a[11], "out_d", M);
    void* const rank = i32(a[12], "out_rank", M);
    return call(entries.build_status, handle(a[0]), act_off, act_prompt, act_gen, act_rem, na, q_off, q_prompt, q_len, nq, finish,
                q_finish, d, rank, stream());
}

struct Requests {
    int64_t n;
    void *ctx0, *len, *budget, *exclude;

    // ctx0, pred_len, budget, exclude_inst
    Requests(PyObject* const* a)
        : n(numel(a[0])), ctx0(i32(a[0], "ctx0")), len(i32(a[1], "pred_len", n)), budget(f32(a[2], "budget", n)),
          exclude(i32(a[3], "exclude_inst", n)) {}
};

struct Choices {
    void *inst, *slack, *fallback;

    // out_inst, out_slack, out_fallback
    Choices(PyObject* const* a, int64_t n)
        : inst(i32(a[0], "out_inst", n)), slack(f32(a[1], "out_slack", n)), fallback(u8(a[2], "out_fallback", n)) {}
};

// n_inst, requests, choices, out_T
PyObject* score_route(PyObject* const* a)
{
    const Requests r(a + 2);
    const Choices c(a + 6, r.n);
    void* const T = f32(a[9], "out_T", r.n * integer(a[1]));
    return call(entries.score_route, handle(a[0]), r.n, r.ctx0, r.len, r.budget, r.exclude, c.inst, c.slack, c.fallback, T, stream());
}

// requests, choices
PyObject* score_route_noalloc(PyObject* const* a)
{
    const Requests r(a + 1);
    const Choices c(a + 5, r.n);
    return call(entries.score_route_noalloc, handle(a[0]), r.n, r.ctx0, r.len, r.budget, r.exclude, c.inst, c.slack, c.fallback, stream());
}

// n_inst, requests, hit_off, hit_inst, hit_len, choices, out_T
PyObject* score_route_cached(PyObject* const* a)
{
    const int64_t nh = numel(a[7]);
    const Requests r(a + 2);
    void* const off = i32(a[6], "hit_off", r.n + 1);
    void* const inst = i32(a[7], "hit_inst");
    void* const len = i32(a[8], "hit_len", nh);
    const Choices c(a + 9, r.n);
    void* const T = f32(a[12], "out_T", r.n * integer(a[1]));
    return call(entries.score_route_cached, handle(a[0]), r.n, r.ctx0, r.len, r.budget, r.exclude, off, inst, len, nh, c.inst, c.slack,
                c.fallback, T, stream());
}

// chunk, requests, choices
PyObject* route_feedback(PyObject* const* a)
{
    const Requests r(a + 2);
    const Choices c(a + 6, r.n);
    return call(entries.route_feedback, handle(a[0]), r.n, integer(a[1]), r.ctx0, r.len, r.budget, r.exclude, c.inst, c.slack, c.fallback,
                stream());
}

// n_inst, act_off, act_prompt, act_gen, act_rem_refreshed, q_off, q_prompt, q_len, act_budget, out_flag, out_finish,
// out_target, out_target_slack, out_n_flagged
PyObject* risk_scan(PyObject* const* a)
{
    const int64_t M = integer(a[1]), na = numel(a[3]), nq = numel(a[7]);
    void* const act_off = i32(a[2], "act_off", M + 1);
    void* const act_prompt = i32(a[3], "act_prompt");
    void* const act_gen = i32(a[4], "act_gen", na);
    void* const act_rem = i32(a[5], "act_rem_refreshed", na);
    void* const q_off = i32(a[6], "q_off", M + 1);
    void* const q_prompt = i32(a[7], "q_prompt");
    void* const q_len = i32(a[8], "q_len", nq);
    void* const budget = f32(a[9], "act_budget", na);
    void* const flag = u8(a[10], "out_flag", na);
    void* const finish = f32(a[11], "out_finish", na);
    void* const target = i32(a[12], "out_target", na);
    void* const slack = f32(a[13], "out_target_slack", na);
    void* const n_flagged = i32(a[14], "out_n_flagged", 1);
    return call(entries.risk_scan, handle(a[0]), act_off, act_prompt, act_gen, act_rem, na, q_off, q_prompt, q_len, nq, budget, flag, finish,
                target, slack, n_flagged, stream());
}

// check_slowly, then the addresses of the entry points in the order of Entries
PyObject* connect(PyObject* const* a)
{
    void** const to = reinterpret_cast<void**>(&entries);
    for (size_t i = 0; i < sizeof entries / sizeof(void*); ++i) to[i] = handle(a[1 + i]);
    Py_INCREF(a[0]);
    Py_XSETREF(check_slowly, a[0]);
    Py_RETURN_NONE;
}

#define GR_METHOD(name, n) {#name, (PyCFunction)(void (*)(void))guarded<n, name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {GR_METHOD(build_status, 13), GR_METHOD(score_route, 10), GR_METHOD(score_route_noalloc, 8),
                         GR_METHOD(score_route_cached, 13), GR_METHOD(route_feedback, 9), GR_METHOD(risk_scan, 15),
                         GR_METHOD(connect, 7), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_goodroute_marshal(void) { return PyModule_Create(&module); }
