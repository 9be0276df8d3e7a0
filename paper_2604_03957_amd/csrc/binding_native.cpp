// The calls of binding.py that a program makes per layer, marshalled in C++: a ctypes call of 10 to 20 arguments takes
// 1.5 to 4 us of Python beside the 2.3 us a kernel launch costs the host, which is what a small layer waits for.
//
// bind(name, address, fallback) returns a function that takes what `fallback` (the Python form of the call) takes.
// The ordinary call -- device tensors, Python integers within the C types, the current stream -- goes straight to
// the C entry point at `address`; any other one (addresses as integers, host tensors, tensor subclasses, wrapped
// tensors, a given stream, numbers of other types, a wrong argument list) is handed to `fallback` unchanged, so what
// such calls do and raise is written in one place.  us per call on the host, ctypes / here: bwta_linear 4.3 / 3.1, the
// eleven calls of a decoder block 53 / 38, the nine of an attention layer 38 / 26.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstdint>
#include <cstring>
#include <new>

#include "../../include/bwta.h"

namespace {

constexpr int kMaxParams = 24;

struct Bound;
// fills the call's arguments from `v` (one slot per parameter, null where not given) and makes it; false: not an
// ordinary call, nothing was done
typedef bool (*Marshal)(const Bound &b, PyObject *const *v, PyObject **result);

struct Spec {
    const char *name;
    int positional;  // parameters before the keyword-only ones
    const char *params[kMaxParams + 1];
    Marshal marshal;
};

struct Bound {
    PyObject_HEAD
    vectorcallfunc call;
    const Spec *spec;
    PyObject *names[kMaxParams];  // interned parameter names
    int count;
    void *address;
    PyObject *fallback;
    PyObject *weak;  // weak references
};

PyObject *g_check = nullptr, *g_raw_stream = nullptr, *g_device = nullptr;  // binding._check, torch's two stream calls

struct NotOrdinary {};

// ---- argument readers: throw NotOrdinary for anything but the ordinary form

const at::Tensor *tensor(PyObject *o)
{
    if (o == nullptr || o == Py_None) return nullptr;
    if (!THPVariable_CheckExact(o)) throw NotOrdinary{};
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda()) throw NotOrdinary{};
    return &t;
}

void *address(const at::Tensor *t) { return t ? t->data_ptr() : nullptr; }  // throws for tensors without storage

int64_t int64(PyObject *o)
{
    if (o == nullptr || !PyLong_CheckExact(o)) throw NotOrdinary{};
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow) throw NotOrdinary{};
    return v;
}

int int32(PyObject *o)
{
    const int64_t v = int64(o);
    if (v < INT_MIN || v > INT_MAX) throw NotOrdinary{};
    return (int)v;
}

bool given(PyObject *o) { return o != nullptr && o != Py_None; }
int64_t int64_or(PyObject *o, int64_t otherwise) { return given(o) ? int64(o) : otherwise; }

int scale_mode(PyObject *o, const at::Tensor *s)
{
    if (given(o)) return int32(o);
    return s == nullptr ? BWTA_SCALE_NONE : s->numel() == 1 ? BWTA_SCALE_SCALAR : BWTA_SCALE_VECTOR;
}

size_t bytes_of(PyObject *o, const at::Tensor *t)
{
    if (!given(o)) return t ? t->nbytes() : 0;
    const int64_t v = int64(o);
    if (v < 0) throw NotOrdinary{};
    return (size_t)v;
}

float number(PyObject *o, float otherwise)
{
    if (o == nullptr) return otherwise;
    if (!PyFloat_CheckExact(o)) throw NotOrdinary{};
    return (float)PyFloat_AS_DOUBLE(o);
}

// the current stream of the current device, as binding._stream finds it
void *current_stream(PyObject *o)
{
    if (given(o)) throw NotOrdinary{};
    PyObject *device = PyObject_CallNoArgs(g_device);
    PyObject *raw = device ? PyObject_CallOneArg(g_raw_stream, device) : nullptr;
    Py_XDECREF(device);
    void *st = raw ? PyLong_AsVoidPtr(raw) : nullptr;
    Py_XDECREF(raw);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        throw NotOrdinary{};
    }
    return st;
}

// the C call without the interpreter lock (a launch waits where the queue is full), its code turned into what the Python
// form returns or raises
template <typename F>
bool finish(F f, PyObject **result, const int *value = nullptr)
{
    int code;
    Py_BEGIN_ALLOW_THREADS
    code = f();
    Py_END_ALLOW_THREADS
    if (code != BWTA_OK) {
        PyObject *c = PyLong_FromLong(code);
        PyObject *r = c ? PyObject_CallOneArg(g_check, c) : nullptr;  // raises
        Py_XDECREF(c);
        Py_XDECREF(r);
        *result = nullptr;
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "bwta call failed");
        return true;
    }
    if (value) {
        *result = PyLong_FromLong(*value);
    } else {
        Py_INCREF(Py_None);
        *result = Py_None;
    }
    return true;
}

#define BWTA_FN(fn) auto *call = (decltype(&fn))b.address

bool linear(const Bound &b, PyObject *const *v, PyObject **result)
{
    const at::Tensor *A = tensor(v[0]), *s_a = tensor(v[1]), *w = tensor(v[2]), *s_w = tensor(v[3]), *out = tensor(v[4]), *ws = tensor(v[5]);
    const int M = int32(v[6]), N = int32(v[7]), K = int32(v[8]);
    const int64_t lda = int64_or(v[9], K), ldo = int64_or(v[10], N);
    const int am = scale_mode(v[11], s_a), wm = scale_mode(v[12], s_w);
    const size_t bytes = bytes_of(v[13], ws);
    void *const pA = address(A), *const psa = address(s_a), *const pw = address(w), *const psw = address(s_w), *const po = address(out), *const pws = address(ws);
    void *const st = current_stream(v[14]);
    BWTA_FN(bwta_linear);
    return finish([&] { return call(pA, lda, psa, am, (const uint32_t *)pw, psw, wm, M, N, K, po, ldo, pws, bytes, st); }, result);
}

bool gemm(const Bound &b, PyObject *const *v, PyObject **result)
{
    const at::Tensor *mask = tensor(v[0]), *sign = tensor(v[1]), *w = tensor(v[2]), *s_a = tensor(v[3]), *s_w = tensor(v[4]), *acc = tensor(v[5]),
                     *out = tensor(v[6]), *ws = tensor(v[7]);
    const int M = int32(v[8]), N = int32(v[9]), K = int32(v[10]);
    const int64_t ldo = int64_or(v[11], N);
    const int am = scale_mode(v[12], s_a), wm = scale_mode(v[13], s_w);
    const size_t bytes = bytes_of(v[14], ws);
    void *const pm = address(mask), *const ps = address(sign), *const pw = address(w), *const psa = address(s_a), *const psw = address(s_w),
               *const pacc = address(acc), *const po = address(out), *const pws = address(ws);
    void *const st = current_stream(v[15]);
    BWTA_FN(bwta_gemm);
    return finish([&] { return call((const uint32_t *)pm, (const uint32_t *)ps, (const uint32_t *)pw, M, N, K, psa, am, psw, wm, (int32_t *)pacc, po, ldo, pws, bytes, st); }, result);
}

bool gemm_prepared(const Bound &b, PyObject *const *v, PyObject **result)
{
    const at::Tensor *prep = tensor(v[0]), *w = tensor(v[1]), *s_a = tensor(v[2]), *s_w = tensor(v[3]), *acc = tensor(v[4]), *out = tensor(v[5]);
    const int fmt = int32(v[6]), M = int32(v[7]), N = int32(v[8]), K = int32(v[9]);
    const int64_t ldo = int64_or(v[10], N);
    const int am = scale_mode(v[11], s_a), wm = scale_mode(v[12], s_w);
    const size_t bytes = bytes_of(v[13], prep);
    void *const pp = address(prep), *const pw = address(w), *const psa = address(s_a), *const psw = address(s_w), *const pacc = address(acc), *const po = address(out);
    void *const st = current_stream(v[14]);
    BWTA_FN(bwta_gemm_prepared);
    return finish([&] { return call(pp, bytes, fmt, (const uint32_t *)pw, M, N, K, psa, am, psw, wm, (int32_t *)pacc, po, ldo, st); }, result);
}

bool prepare_act(const Bound &b, PyObject *const *v, PyObject **result)
{
    const at::Tensor *A = tensor(v[0]), *s_a = tensor(v[1]), *prep = tensor(v[2]);
    const int M = int32(v[3]), K = int32(v[4]);
    const int64_t lda = int64_or(v[5], K);
    const int am = scale_mode(v[6], s_a);
    const size_t bytes = bytes_of(v[7], prep);
    void *const pA = address(A), *const psa = address(s_a), *const pp = address(prep);
    void *const st = current_stream(v[8]);
    int fmt = 0;
    BWTA_FN(bwta_prepare_act);
    return finish([&] { return call(pA, lda, psa, am, M, K, pp, bytes, &fmt, st); }, result, &fmt);
}

bool prepare_act_autoscale(const Bound &b, PyObject *const *v, PyObject **result)
{
    const at::Tensor *A = tensor(v[0]), *s_a = tensor(v[1]), *prep = tensor(v[2]);
    const int M = int32(v[3]), K = int32(v[4]);
    const int64_t lda = int64_or(v[5], K);
    const size_t bytes = bytes_of(v[6], prep);
    void *const pA = address(A), *const psa = address(s_a), *const pp = address(prep);
    void *const st = current_stream(v[7]);
    int fmt = 0;
    BWTA_FN(bwta_prepare_act_autoscale);
    return finish([&] { return call(pA, lda, M, K, psa, pp, bytes, &fmt, st); }, result, &fmt);
}

bool quantize_pack_act(const Bound &b, PyObject *const *v, PyObject **result)
{
    const at::Tensor *A = tensor(v[0]), *s_a = tensor(v[1]), *mask = tensor(v[2]), *sign = tensor(v[3]), *nnz = tensor(v[4]);
    const int M = int32(v[5]), K = int32(v[6]);
    const int64_t lda = int64_or(v[7], K);
    const int dtype = v[8] ? int32(v[8]) : BWTA_DTYPE_FP16;
    const int am = scale_mode(v[9], s_a);
    void *const pA = address(A), *const psa = address(s_a), *const pm = address(mask), *const ps = address(sign), *const pn = address(nnz);
    void *const st = current_stream(v[10]);
    BWTA_FN(bwta_quantize_pack_act);
    return finish([&] { return call(pA, dtype, lda, psa, am, M, K, (uint32_t *)pm, (uint32_t *)ps, (int32_t *)pn, st); }, result);
}

bool quantize_pack_bool(const Bound &b, PyObject *const *v, PyObject **result)
{
    const at::Tensor *A = tensor(v[0]), *s_a = tensor(v[1]), *mask = tensor(v[2]);
    const int M = int32(v[3]), K = int32(v[4]);
    const int64_t lda = int64_or(v[5], K);
    const int am = scale_mode(v[6], s_a);
    void *const pA = address(A), *const psa = address(s_a), *const pm = address(mask);
    void *const st = current_stream(v[7]);
    BWTA_FN(bwta_quantize_pack_bool);
    return finish([&] { return call(pA, lda, psa, am, M, K, (uint32_t *)pm, st); }, result);
}

bool act_scale(const Bound &b, PyObject *const *v, PyObject **result)
{
    const at::Tensor *A = tensor(v[0]), *s = tensor(v[1]);
    const int M = int32(v[2]), K = int32(v[3]);
    const int64_t lda = int64_or(v[4], K);
    void *const pA = address(A), *const ps = address(s);
    void *const st = current_stream(v[5]);
    BWTA_FN(bwta_act_scale);
    return finish([&] { return call(pA, lda, M, K, ps, st); }, result);
}

bool prepare_weights(const Bound &b, PyObject *const *v, PyObject **result)
{
    const at::Tensor *W = tensor(v[0]), *w = tensor(v[1]), *s_w = tensor(v[2]);
    const int N = int32(v[3]), K = int32(v[4]);
    const int64_t ldw = int64_or(v[5], K);
    void *const pW = address(W), *const pw = address(w), *const psw = address(s_w);
    void *const st = current_stream(v[6]);
    BWTA_FN(bwta_prepare_weights);
    return finish([&] { return call(pW, ldw, N, K, (uint32_t *)pw, psw, st); }, result);
}

int64_t row_words(int K) { return 4 * (((int64_t)K + 127) / 128); }  // bwta_plane_row_words of a positive K

bool matmul_tt(const Bound &b, PyObject *const *v, PyObject **result)
{
    const at::Tensor *ma = tensor(v[0]), *sa = tensor(v[1]), *mb = tensor(v[2]), *sb = tensor(v[3]), *s_a = tensor(v[4]), *s_b = tensor(v[5]),
                     *acc = tensor(v[6]), *out = tensor(v[7]);
    const int batch = int32(v[8]), M = int32(v[9]), N = int32(v[10]), K = int32(v[11]);
    if (M <= 0 || N <= 0 || K <= 0) throw NotOrdinary{};
    const float alpha = number(v[12], 1.0f);
    const int64_t strideA = int64_or(v[13], M * row_words(K)), strideB = int64_or(v[14], N * row_words(K)), ldo = int64_or(v[15], N);
    if (ldo < 0 || ldo > INT_MAX) throw NotOrdinary{};
    const int64_t stride_out = int64_or(v[16], M * ldo);
    const int am = scale_mode(v[17], s_a), bm = scale_mode(v[18], s_b);
    void *const pma = address(ma), *const psa = address(sa), *const pmb = address(mb), *const psb = address(sb), *const pa = address(s_a), *const pb = address(s_b),
               *const pacc = address(acc), *const po = address(out);
    void *const st = current_stream(v[19]);
    BWTA_FN(bwta_matmul_tt);
    return finish([&] { return call((const uint32_t *)pma, (const uint32_t *)psa, strideA, (const uint32_t *)pmb, (const uint32_t *)psb, strideB, batch, M, N, K, pa, am, pb, bm,
                                    alpha, (int32_t *)pacc, po, ldo, stride_out, st); }, result);
}

bool matmul_bool_prepared(const Bound &b, PyObject *const *v, PyObject **result)
{
    const at::Tensor *ma = tensor(v[0]), *prep = tensor(v[1]), *s_a = tensor(v[2]), *s_b = tensor(v[3]), *out = tensor(v[4]);
    const int fmt = int32(v[5]), batch = int32(v[6]), M = int32(v[7]), N = int32(v[8]), K = int32(v[9]);
    if (M <= 0 || N <= 0 || K <= 0) throw NotOrdinary{};
    const float alpha = number(v[10], 1.0f);
    const int64_t strideA = int64_or(v[11], M * row_words(K)), ldo = int64_or(v[12], N);
    if (ldo < 0 || ldo > INT_MAX) throw NotOrdinary{};
    const int64_t stride_out = int64_or(v[13], M * ldo);
    const int am = scale_mode(v[14], s_a), bm = scale_mode(v[15], s_b);
    const size_t bytes = bytes_of(v[16], prep);
    void *const pma = address(ma), *const pp = address(prep), *const pa = address(s_a), *const pb = address(s_b), *const po = address(out);
    void *const st = current_stream(v[17]);
    BWTA_FN(bwta_matmul_bool_prepared);
    return finish([&] { return call((const uint32_t *)pma, strideA, pp, bytes, fmt, batch, M, N, K, pa, am, pb, bm, alpha, po, ldo, stride_out, st); }, result);
}

const Spec kSpecs[] = {
    {"bwta_linear", 6, {"A", "s_a", "wsign", "s_w", "out", "workspace", "M", "N", "K", "lda", "ldo", "a_scale_mode", "w_scale_mode", "workspace_bytes", "stream"}, linear},
    {"bwta_gemm", 8, {"mask", "sign", "wsign", "s_a", "s_w", "acc", "out", "workspace", "M", "N", "K", "ldo", "a_scale_mode", "w_scale_mode", "workspace_bytes", "stream"}, gemm},
    {"bwta_gemm_prepared", 6, {"prepared", "wsign", "s_a", "s_w", "acc", "out", "fmt", "M", "N", "K", "ldo", "a_scale_mode", "w_scale_mode", "prepared_bytes", "stream"}, gemm_prepared},
    {"bwta_prepare_act", 3, {"A", "s_a", "prepared", "M", "K", "lda", "a_scale_mode", "prepared_bytes", "stream"}, prepare_act},
    {"bwta_prepare_act_autoscale", 3, {"A", "s_a", "prepared", "M", "K", "lda", "prepared_bytes", "stream"}, prepare_act_autoscale},
    {"bwta_quantize_pack_act", 5, {"A", "s_a", "mask", "sign", "nnz", "M", "K", "lda", "a_dtype", "scale_mode", "stream"}, quantize_pack_act},
    {"bwta_quantize_pack_bool", 3, {"A", "s_a", "mask", "M", "K", "lda", "scale_mode", "stream"}, quantize_pack_bool},
    {"bwta_act_scale", 2, {"A", "s", "M", "K", "lda", "stream"}, act_scale},
    {"bwta_prepare_weights", 3, {"W", "wsign", "s_w", "N", "K", "ldw", "stream"}, prepare_weights},
    {"bwta_matmul_tt", 8, {"maskA", "signA", "maskB", "signB", "s_a", "s_b", "acc", "out", "batch", "M", "N", "K", "alpha", "strideA", "strideB", "ldo", "stride_out", "a_scale_mode", "b_scale_mode", "stream"}, matmul_tt},
    {"bwta_matmul_bool_prepared", 5, {"maskA", "preparedB", "s_a", "s_b", "out", "fmt", "batch", "M", "N", "K", "alpha", "strideA", "ldo", "stride_out", "a_scale_mode", "b_scale_mode", "prepared_bytes", "stream"}, matmul_bool_prepared},
};

// the arguments to their parameters' slots; false where the Python form would raise or this table does not know better
bool place(const Bound &b, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames, PyObject **v)
{
    if (nargs > b.spec->positional) return false;
    for (int i = 0; i < b.count; ++i) v[i] = i < nargs ? args[i] : nullptr;
    const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    int at = (int)nargs;
    for (Py_ssize_t k = 0; k < nkw; ++k) {
        PyObject *name = PyTuple_GET_ITEM(kwnames, k);
        int i = 0;
        for (; i < b.count; ++i, at = at + 1 < b.count ? at + 1 : 0)  // names come in order as a rule, and interned
            if (b.names[at] == name) break;
        if (i == b.count || v[at]) return false;
        v[at] = args[nargs + k];
    }
    // the tensors all have to be given, except nnz, which may be left out
    for (int i = 0; i < b.spec->positional; ++i)
        if (!v[i] && strcmp(b.spec->params[i], "nnz") != 0) return false;
    return true;
}

PyObject *bound_call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames)
{
    const Bound &b = *(const Bound *)self;
    PyObject *v[kMaxParams], *result = nullptr;
    if (place(b, args, PyVectorcall_NARGS(nargsf), kwnames, v)) {
        try {
            if (b.spec->marshal(b, v, &result)) return result;
        } catch (const std::bad_alloc &) {
            return PyErr_NoMemory();
        } catch (...) {  // not the ordinary form, or a tensor without an address: the Python form's business
            PyErr_Clear();
        }
    }
    return PyObject_Vectorcall(b.fallback, args, nargsf & ~PY_VECTORCALL_ARGUMENTS_OFFSET, kwnames);
}

void bound_dealloc(PyObject *self)
{
    Bound *b = (Bound *)self;
    if (b->weak) PyObject_ClearWeakRefs(self);
    for (int i = 0; i < b->count; ++i) Py_XDECREF(b->names[i]);
    Py_XDECREF(b->fallback);
    Py_TYPE(self)->tp_free(self);
}

// Everything a program may do with a Python function besides calling it: its attributes, __class__ among them, are those
// of the Python form and are set there, it binds as a method, and is pickled and copied by its name.
PyObject *bound_getattro(PyObject *self, PyObject *name)
{
    if (PyUnicode_Check(name)) {
        const char *s = PyUnicode_AsUTF8(name);
        if (!s) return nullptr;
        if (strcmp(s, "__reduce_ex__") == 0 || strcmp(s, "__reduce__") == 0 || strcmp(s, "__get__") == 0) return PyObject_GenericGetAttr(self, name);
    }
    return PyObject_GetAttr(((Bound *)self)->fallback, name);
}

int bound_setattro(PyObject *self, PyObject *name, PyObject *value) { return PyObject_SetAttr(((Bound *)self)->fallback, name, value); }

PyObject *bound_descr_get(PyObject *self, PyObject *object, PyObject *)
{
    if (object == nullptr || object == Py_None) {
        Py_INCREF(self);
        return self;
    }
    return PyMethod_New(self, object);
}

PyObject *bound_repr(PyObject *self) { return PyObject_Repr(((Bound *)self)->fallback); }

PyObject *bound_reduce(PyObject *self, PyObject *) { return PyObject_GetAttrString(((Bound *)self)->fallback, "__qualname__"); }

PyMethodDef kBoundMethods[] = {{"__reduce_ex__", bound_reduce, METH_O, nullptr}, {"__reduce__", bound_reduce, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};

PyTypeObject BoundType = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject *bind(PyObject *, PyObject *args)
{
    const char *name;
    PyObject *addr, *fallback;
    if (!PyArg_ParseTuple(args, "sOO", &name, &addr, &fallback)) return nullptr;
    for (const Spec &s : kSpecs) {
        if (strcmp(s.name, name) != 0) continue;
        void *const address = PyLong_AsVoidPtr(addr);
        if (PyErr_Occurred()) return nullptr;
        Bound *b = PyObject_New(Bound, &BoundType);
        if (!b) return nullptr;
        b->call = bound_call, b->spec = &s, b->count = 0, b->address = address, b->fallback = fallback, b->weak = nullptr;
        Py_INCREF(fallback);
        for (; s.params[b->count]; ++b->count) {
            b->names[b->count] = PyUnicode_InternFromString(s.params[b->count]);
            if (!b->names[b->count]) {
                Py_DECREF(b);
                return nullptr;
            }
        }
        return (PyObject *)b;
    }
    PyErr_Format(PyExc_KeyError, "%s", name);
    return nullptr;
}

PyObject *setup(PyObject *, PyObject *args)  // (check, raw_stream, device)
{
    PyObject *c, *r, *d;
    if (!PyArg_ParseTuple(args, "OOO", &c, &r, &d)) return nullptr;
    Py_INCREF(c), Py_INCREF(r), Py_INCREF(d);
    Py_XDECREF(g_check), Py_XDECREF(g_raw_stream), Py_XDECREF(g_device);
    g_check = c, g_raw_stream = r, g_device = d;
    Py_RETURN_NONE;
}

PyObject *parameters(PyObject *, PyObject *)  // {name: (positional parameters, all parameters)}
{
    PyObject *out = PyDict_New();
    for (const Spec &s : kSpecs) {
        PyObject *l = out ? PyList_New(0) : nullptr;
        if (!l) break;
        for (int i = 0; s.params[i]; ++i) {
            PyObject *p = PyUnicode_FromString(s.params[i]);
            if (p) PyList_Append(l, p);
            Py_XDECREF(p);
        }
        PyObject *t = Py_BuildValue("(iN)", s.positional, l);
        if (t) PyDict_SetItemString(out, s.name, t);
        Py_XDECREF(t);
    }
    if (PyErr_Occurred()) {
        Py_XDECREF(out);
        return nullptr;
    }
    return out;
}

#ifndef BWTA_IDENTITY
#define BWTA_IDENTITY "unknown"
#endif
PyObject *identity(PyObject *, PyObject *) { return PyUnicode_FromString(BWTA_IDENTITY); }

PyMethodDef kMethods[] = {{"identity", identity, METH_NOARGS, "identity() -> \"<digest of the sources> <torch version> <Python version>\""},
                          {"bind", bind, METH_VARARGS, "bind(name, address, fallback) -> function"},
                          {"setup", setup, METH_VARARGS, "setup(check, raw_stream, device)"},
                          {"parameters", parameters, METH_NOARGS, "{name: (positional parameters, all parameters)}"},
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_bwta_native", "Marshalling of the per-layer calls.", -1, kMethods};

}  // namespace

PyMODINIT_FUNC PyInit__bwta_native(void)
{
#define BWTA_STR2(x) #x
#define BWTA_STR(x) BWTA_STR2(x)
    constexpr char built_for[] = BWTA_STR(PY_MAJOR_VERSION) "." BWTA_STR(PY_MINOR_VERSION) ".";
    if (strncmp(Py_GetVersion(), built_for, sizeof built_for - 1) != 0) {
        PyErr_SetString(PyExc_ImportError, "built for another version of Python");
        return nullptr;
    }
    BoundType.tp_name = "_bwta_native.function";
    BoundType.tp_basicsize = sizeof(Bound);
    BoundType.tp_dealloc = bound_dealloc;
    BoundType.tp_call = PyVectorcall_Call;
    BoundType.tp_vectorcall_offset = offsetof(Bound, call);
    BoundType.tp_getattro = bound_getattro;
    BoundType.tp_setattro = bound_setattro;
    BoundType.tp_descr_get = bound_descr_get;
    BoundType.tp_repr = bound_repr;
    BoundType.tp_methods = kBoundMethods;
    BoundType.tp_weaklistoffset = offsetof(Bound, weak);
    BoundType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL;
    if (PyType_Ready(&BoundType) < 0) return nullptr;
    return PyModule_Create(&kModule);
}
