// The calls of the Python binding that a decode step or a small product makes, without an interpreter between the tensors and the C ABI.
//
// A single product from Python was bound by its marshalling: attribute look-ups on tensors, checks and the conversion of thirteen
// arguments took 2 to 3 us of a call whose kernel takes 2 to 5.  Here an argument is looked at where it lies, in the tensor's own structure: W1A2 16 x 256 x 512
// (pack + product) 10.9 -> 8.2 us, W2A2 1 x 11008 x 4096 from codes 6.2 -> 4.6, of which the kernel takes 4.4.  Outputs that are not given are allocated here:
// handed over, such a call took 0.1 to 0.3 us longer than without this module (W2A2 1 x 1024 x 1024 6.9 -> 7.1 us, from codes 7.3 -> 7.6, quantisation 6.7 -> 7.0), now 5.0, 5.0 and 4.5.
//
// Every function takes the arguments of the Python function of the same name in binding.py and has that function as its `general` form: whatever
// is not the plain case (anything that is not a torch.Tensor, an integer of another type, an output that cannot be allocated, a check
// that fails, an unknown keyword, a torch-function mode, a process forked from one that uses the GPU, the library not loaded yet) is handed to it with the very arguments, so that
// results and errors are its own.  A status other than 0 goes to binding.py's _check, on the same thread.  As through ctypes, the interpreter's lock is
// released around the call.
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/device_lazy_init.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>

#include <cstring>

#include "../../include/apmm.h"
#include "apmm_call_guard.h"

namespace {

struct Library {
    decltype(&apmm_packed_bytes) packed_bytes;
    decltype(&apmm_packed_activation_bytes) packed_activation_bytes;
    decltype(&apmm_pack_weights) pack_weights;
    decltype(&apmm_pack_activations) pack_activations;
    decltype(&apmm_quantize_pack_activations) quantize_pack_activations;
    decltype(&apmm_gemm_ex) gemm_ex;
    decltype(&apmm_gemm_from_codes) gemm_from_codes;
};
Library lib = {};
bool loaded = false;
PyObject *check = nullptr;  // binding.py's _check

constexpr int kMaxArgs = 15;
enum Function { kPackWeights, kPackActivations, kQuantize, kGemm, kFromCodes, kFunctions };
struct Signature {
    const char *name;
    int count, required;
    const char *args[kMaxArgs];
    PyObject *keys[kMaxArgs];  // the interned names
    PyObject *general;
};
Signature signatures[kFunctions] = {
    {"apmm_pack_weights", 3, 2, {"w_codes", "q", "out"}, {}, nullptr},
    {"apmm_pack_activations", 3, 2, {"a_codes", "p", "out"}, {}, nullptr},
    {"apmm_quantize_pack_activations", 4, 2, {"x_f16", "p", "out", "scale_out"}, {}, nullptr},
    {"apmm_gemm", 15, 7,
     {"M", "N", "K", "p", "q", "a_packed", "w_packed", "want_i32", "want_f16", "w_scale", "a_scale", "c_i32", "c_f16", "workspace", "algo"}, {}, nullptr},
    {"apmm_gemm_from_codes", 12, 5, {"a_codes", "N", "p", "q", "w_packed", "want_i32", "want_f16", "w_scale", "a_scale", "c_i32", "c_f16", "workspace"}, {}, nullptr},
};

// Arguments by place, null where not given; false: not the plain case.
bool place(const Signature &s, PyObject *const *args, Py_ssize_t nargs, PyObject *names, PyObject **out)
{
    if (!loaded || nargs > s.count || at::impl::torch_function_mode_enabled() || torch::utils::is_device_in_bad_fork(at::kCUDA)) return false;
    for (int i = 0; i < s.count; ++i) out[i] = i < nargs ? args[i] : nullptr;
    const Py_ssize_t named = names ? PyTuple_GET_SIZE(names) : 0;
    for (Py_ssize_t i = 0; i < named; ++i) {
        PyObject *key = PyTuple_GET_ITEM(names, i);
        int at = (int)nargs;
        while (at < s.count && s.keys[at] != key) ++at;
        if (at == s.count || out[at]) return false;
        out[at] = args[nargs + i];
    }
    for (int i = 0; i < s.required; ++i)
        if (!out[i]) return false;
    return true;
}

bool integer(PyObject *o, int64_t lo, int64_t hi, int64_t &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return !overflow && v >= lo && v <= hi;
}
constexpr int64_t kAny = INT64_MAX;

bool flag(PyObject *o, bool absent, bool &v)
{
    v = o ? o == Py_True : absent;
    return !o || o == Py_True || o == Py_False;
}

bool given(PyObject *o) { return o && o != Py_None; }
const at::Tensor *tensor(PyObject *o)
{
    if (!given(o) || !THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() ? &t : nullptr;
}
// null pointer for an absent tensor; false: not the plain case
bool address(PyObject *o, void *&p)
{
    p = nullptr;
    if (!given(o)) return true;
    const at::Tensor *t = tensor(o);
    if (t) p = t->data_ptr();
    return t != nullptr;
}
bool matrix(const at::Tensor *t, at::ScalarType type) { return t && t->scalar_type() == type && t->dim() == 2 && t->is_contiguous(); }
bool scale_ok(PyObject *o, int64_t n)
{
    if (!given(o)) return true;
    const at::Tensor *t = tensor(o);
    return t && t->scalar_type() == at::kHalf && t->numel() == n && t->is_contiguous();
}
size_t bytes(const at::Tensor &t) { return t.nbytes(); }
void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

PyObject *general(const Signature &s, PyObject *const *args, Py_ssize_t nargs, PyObject *names)
{
    if (!s.general) {
        PyErr_SetString(PyExc_RuntimeError, "apmm: the general function is not set");
        return nullptr;
    }
    return PyObject_Vectorcall(s.general, args, (size_t)nargs, names);
}

template <class Call>
bool called(Call call) { return call_and_check(check, call); }

// An output by the place of its argument: the caller's, or a new tensor as the Python function allocates it.  Nothing is given back by a destructor:
// a thread that ends inside the call is unwound without the interpreter's lock.
struct Output {
    PyObject *object = nullptr;  // None where neither given nor wanted
    void *address = nullptr;
    bool made = false;
};
// false: not the plain case
bool output(Output &o, PyObject *arg, bool wanted, const at::Tensor &like, at::IntArrayRef size, at::ScalarType type)
{
    o.object = arg ? arg : Py_None;
    if (given(arg) || !wanted) return address(arg, o.address);
    at::Tensor t;
    bool allocated;
    Py_BEGIN_ALLOW_THREADS
    allocated = end_exceptions([&] { t = at::empty(size, like.options().dtype(type)); return true; }, [] { return false; });
    Py_END_ALLOW_THREADS
    if (!allocated) return false;
    o.object = THPVariable_Wrap(std::move(t));
    o.made = o.object != nullptr;
    if (!o.made) {
        PyErr_Clear();
        return false;
    }
    return address(o.object, o.address);
}
// The result of a call that went well (one output, or two as a tuple), or what stands for one that did not: 1 and the result, else `done`
int result_of(int done, Output &a, Output *b, PyObject *&result)
{
    if (done == 1) {
        result = b ? PyTuple_Pack(2, a.object, b->object) : a.object;
        if (!b) Py_INCREF(result);
        if (!result) done = -1;
    }
    if (a.made) Py_DECREF(a.object);
    if (b && b->made) Py_DECREF(b->object);
    return done;
}
int64_t at_least_one(size_t n) { return n > 1 ? (int64_t)n : 1; }

// Each returns 1 and the result, 0 for the general form, -1 with an error set.
int pack(Function f, PyObject **v, PyObject *&result)
{
    int64_t bits;
    const at::Tensor *codes = tensor(v[0]);
    if (!matrix(codes, at::kByte) || !integer(v[1], 1, 8, bits) || (given(v[2]) && !tensor(v[2]))) return 0;
    const int64_t rows = codes->size(0), K = codes->size(1);
    const bool weights = f == kPackWeights;
    const size_t need = (weights ? lib.packed_bytes : lib.packed_activation_bytes)(rows, K, (int)bits);
    if (given(v[2]) && bytes(*tensor(v[2])) < need) return 0;
    const uint8_t *src = static_cast<const uint8_t *>(codes->data_ptr());
    Output out;
    if (!output(out, v[2], true, *codes, {at_least_one(need)}, at::kByte)) return result_of(0, out, nullptr, result);
    void *s = stream();
    const bool went = called([&] { return (weights ? lib.pack_weights : lib.pack_activations)(src, rows, K, (int)bits, out.address, s); });
    return result_of(went ? 1 : -1, out, nullptr, result);
}

int quantize(PyObject **v, PyObject *&result)
{
    int64_t p;
    const at::Tensor *x = tensor(v[0]);
    if (!matrix(x, at::kHalf) || !integer(v[1], 1, 8, p) || (given(v[2]) && !tensor(v[2])) || (given(v[3]) && !tensor(v[3]))) return 0;
    const int64_t M = x->size(0), K = x->size(1);
    const size_t need = lib.packed_activation_bytes(M, K, (int)p);
    if (given(v[2]) && bytes(*tensor(v[2])) < need) return 0;
    if (given(v[3]) && (tensor(v[3])->scalar_type() != at::kHalf || tensor(v[3])->numel() < M)) return 0;
    const uint16_t *src = static_cast<const uint16_t *>(x->data_ptr());
    Output out, scale;
    if (!output(out, v[2], true, *x, {at_least_one(need)}, at::kByte) || !output(scale, v[3], true, *x, {M}, at::kHalf)) return result_of(0, out, &scale, result);
    void *s = stream();
    const bool went = called([&] { return lib.quantize_pack_activations(src, M, K, (int)p, out.address, static_cast<uint16_t *>(scale.address), s); });
    return result_of(went ? 1 : -1, out, &scale, result);
}

int gemm(PyObject **v, PyObject *&result)
{
    int64_t M, N, K, p, q, algo = APMM_ALGO_AUTO;
    bool want_i32, want_f16;
    void *a, *w, *ws, *as, *space;
    if (!integer(v[0], 0, kAny, M) || !integer(v[1], 0, kAny, N) || !integer(v[2], 0, kAny, K) || !integer(v[3], 0, 255, p) || !integer(v[4], 0, 255, q) ||
        !flag(v[7], true, want_i32) || !flag(v[8], false, want_f16) || !given(v[5]) || !given(v[6]) || (v[14] && !integer(v[14], 0, 255, algo)) ||
        !scale_ok(v[9], N) || !scale_ok(v[10], M) || !address(v[5], a) || !address(v[6], w) || !address(v[9], ws) || !address(v[10], as) || !address(v[13], space))
        return 0;
    const size_t room = given(v[13]) ? bytes(*tensor(v[13])) : 0;
    const at::Tensor &like = *tensor(v[5]);
    Output ci, cf;
    if (!output(ci, v[11], want_i32, like, {M, N}, at::kInt) || !output(cf, v[12], want_f16, like, {M, N}, at::kHalf)) return result_of(0, ci, &cf, result);
    void *s = stream();
    const bool went = called([&] {
        return lib.gemm_ex(M, N, K, (int)p, (int)q, a, w, static_cast<int32_t *>(ci.address), static_cast<uint16_t *>(cf.address), static_cast<const uint16_t *>(ws),
                           static_cast<const uint16_t *>(as), space, room, s, (int)algo);
    });
    return result_of(went ? 1 : -1, ci, &cf, result);
}

int from_codes(PyObject **v, PyObject *&result)
{
    int64_t N, p, q;
    bool want_i32, want_f16;
    void *w, *ws, *as, *space;
    const at::Tensor *codes = tensor(v[0]);
    if (!matrix(codes, at::kByte) || !integer(v[1], 0, kAny, N) || !integer(v[2], 0, 255, p) || !integer(v[3], 0, 255, q) || !given(v[4]) ||
        !flag(v[5], true, want_i32) || !flag(v[6], false, want_f16) || !address(v[4], w) || !address(v[7], ws) || !address(v[8], as) || !address(v[11], space))
        return 0;
    const int64_t M = codes->size(0), K = codes->size(1);
    const uint8_t *a = static_cast<const uint8_t *>(codes->data_ptr());
    const size_t room = given(v[11]) ? bytes(*tensor(v[11])) : 0;
    Output ci, cf;
    if (!output(ci, v[9], want_i32, *codes, {M, N}, at::kInt) || !output(cf, v[10], want_f16, *codes, {M, N}, at::kHalf)) return result_of(0, ci, &cf, result);
    void *s = stream();
    const bool went = called([&] {
        return lib.gemm_from_codes(M, N, K, (int)p, (int)q, a, w, static_cast<int32_t *>(ci.address), static_cast<uint16_t *>(cf.address), static_cast<const uint16_t *>(ws),
                                   static_cast<const uint16_t *>(as), space, room, s);
    });
    return result_of(went ? 1 : -1, ci, &cf, result);
}

template <Function F>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *names)
{
    const Signature &s = signatures[F];
    PyObject *v[kMaxArgs], *result = nullptr;
    const int done = end_exceptions(
        [&] {
            if (!place(s, args, nargs, names, v)) return 0;
            return F <= kPackActivations ? pack(F, v, result) : F == kQuantize ? quantize(v, result) : F == kGemm ? gemm(v, result) : from_codes(v, result);
        },
        [] { return 0; });  // (torch's own refusal of a tensor: the general form meets the same one and reports it)
    if (done > 0) return result;
    return done < 0 ? nullptr : general(s, args, nargs, names);
}

// set_library(addresses of the seven functions in Library's order, _check)
PyObject *set_library(PyObject *, PyObject *args)
{
    unsigned long long at[7];
    PyObject *fn;
    if (!PyArg_ParseTuple(args, "(KKKKKKK)O", &at[0], &at[1], &at[2], &at[3], &at[4], &at[5], &at[6], &fn)) return nullptr;
    static_assert(sizeof(lib) == sizeof(at), "seven functions");
    std::memcpy(&lib, at, sizeof(at));
    Py_INCREF(fn);
    Py_XDECREF(check);
    check = fn;
    loaded = true;
    Py_RETURN_NONE;
}

// set_general(name, function): the Python function of an entry point
PyObject *set_general(PyObject *, PyObject *args)
{
    const char *name;
    PyObject *fn;
    if (!PyArg_ParseTuple(args, "sO", &name, &fn)) return nullptr;
    for (Signature &s : signatures) {
        if (std::strcmp(s.name, name) != 0) continue;
        Py_INCREF(fn);
        Py_XDECREF(s.general);
        s.general = fn;
        Py_RETURN_NONE;
    }
    PyErr_SetString(PyExc_KeyError, name);
    return nullptr;
}

#define ENTRY(F) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(entry<F>)), METH_FASTCALL | METH_KEYWORDS
PyMethodDef methods[] = {
    {"apmm_pack_weights", ENTRY(kPackWeights),
     "apmm_pack_weights(w_codes, q, out=None)\n--\n\nN x K uint8 weight codes -> opaque packed buffer (uint8 tensor)."},
    {"apmm_pack_activations", ENTRY(kPackActivations),
     "apmm_pack_activations(a_codes, p, out=None)\n--\n\nM x K uint8 activation codes -> opaque packed buffer (uint8 tensor)."},
    {"apmm_quantize_pack_activations", ENTRY(kQuantize),
     "apmm_quantize_pack_activations(x_f16, p, out=None, scale_out=None)\n--\n\nM x K float16 activations -> (opaque packed buffer, float16 per-token scales)."},
    {"apmm_gemm", ENTRY(kGemm),
     "apmm_gemm(M, N, K, p, q, a_packed, w_packed, want_i32=True, want_f16=False, w_scale=None, a_scale=None, c_i32=None, c_f16=None, workspace=None, "
     "algo=0)\n--\n\nC = A W^T on packed operands.  Returns (c_i32 or None, c_f16 or None)."},
    {"apmm_gemm_from_codes", ENTRY(kFromCodes),
     "apmm_gemm_from_codes(a_codes, N, p, q, w_packed, want_i32=True, want_f16=False, w_scale=None, a_scale=None, c_i32=None, c_f16=None, "
     "workspace=None)\n--\n\nC = A W^T straight from the M x K uint8 activation codes."},
    {"set_library", set_library, METH_VARARGS, nullptr},
    {"set_general", set_general, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "paper_2409_17870_amd._apmm_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__apmm_call()
{
    for (Signature &s : signatures)
        for (int i = 0; i < s.count; ++i)
            if (!(s.keys[i] = PyUnicode_InternFromString(s.args[i]))) return nullptr;
    return PyModule_Create(&module);
}
