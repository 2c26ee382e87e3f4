// The binding's fast path: argument checks, output allocation and the C call of
// the per-round entry points in native code.
//
// Each function takes the address of the library's entry point and the call's
// arguments, checks them as the Python functions do, and makes the call on the
// current stream.  It returns (accept_len, next_token) or True, or the library's
// status when that is not ASD_OK, or None, with nothing done, for any argument
// that is not the ordinary one (a scalar gate, a tensor on another device, a
// layout to copy, a subclass, a wrong shape, an active dispatch mode): the
// Python function then takes the call, converts or copies what it accepts and
// raises what it refuses.
//
// A call's checks, pointers and outputs in Python took more host time than the
// GPU needs for a small round.  Host time per call of the public functions, before
// and after: one request with 8 drafts of 32,000 logits 15.5 and 5.8 us (3.8 of it
// in this module and the launch; the call itself 15.5 and 7.3 us, now the
// kernel's time); verify with commit 20.0 and 8.2 us; the opportunity statistic
// 12.2 and 3.5 us; the fused output layer 21.9 and 10.5.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/asd.h"

#ifndef ASD_BINDING_HASH
#define ASD_BINDING_HASH "unhashed"
#endif

namespace {

using at::ScalarType;

// A dense GPU tensor of this type on the current device, or nullptr.
const at::Tensor* dense(PyObject* o, ScalarType type, int device) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || !t.has_storage() ||
        t.get_device() != device || t.scalar_type() != type || !t.is_contiguous())
        return nullptr;
    return &t;
}

// Pointer of a vector of `n` elements (any length for n < 0); false if it is
// not one.  None gives nullptr where `optional`.
bool vec(PyObject* o, ScalarType type, int64_t n, int device, void** out, bool optional = false) {
    *out = nullptr;
    if (o == Py_None) return optional;
    const at::Tensor* t = dense(o, type, device);
    if (!t || t->dim() != 1 || (n >= 0 && t->size(0) != n)) return false;
    *out = t->data_ptr();
    return true;
}

int current_device(PyObject* o) {
    if (c10::impl::TorchDispatchModeTLS::any_modes_set() || !THPVariable_CheckExact(o)) return -1;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda()) return -1;
    const int device = t.get_device();
    return device == c10::hip::current_device() ? device : -1;
}

void* current_stream(int device) {
    return (void*)c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream();
}

// The arguments that every verifying call shares, from args[0]: draft tokens,
// block lengths, gates, caps, ledgers, row offsets, accepted lengths, next
// tokens, argmax, regret.
constexpr int kShared = 10;
struct Shared {
    int32_t n = 0;
    int64_t rows = 0;
    void *draft, *lens, *tau, *cap, *budget, *offsets, *accept, *next, *argmax, *regret;
    void* stream = nullptr;
    PyObject* outputs[2] = {nullptr, nullptr};       // owned references
    at::Tensor fresh[2];

    bool take(PyObject* const* a, int64_t total_rows, int device) {
        rows = total_rows;
        const at::Tensor* l = dense(a[1], ScalarType::Int, device);
        if (!l || l->dim() != 1 || l->size(0) > INT32_MAX) return false;
        n = (int32_t)l->size(0);
        lens = l->data_ptr();
        const at::Tensor* b = dense(a[4], ScalarType::Float, device);
        if (!b || b->dim() != 2 || b->size(0) != n || b->size(1) != 2) return false;
        budget = b->data_ptr();
        if (!vec(a[0], ScalarType::Int, rows, device, &draft) ||
            !vec(a[2], ScalarType::Float, n, device, &tau) ||
            !vec(a[3], ScalarType::Int, n, device, &cap) ||
            !vec(a[5], ScalarType::Long, n, device, &offsets, true) ||
            !vec(a[6], ScalarType::Int, n, device, &accept, true) ||
            !vec(a[7], ScalarType::Int, n, device, &next, true) ||
            !vec(a[8], ScalarType::Int, rows, device, &argmax, true) ||
            !vec(a[9], ScalarType::Float, rows, device, &regret, true))
            return false;
        void** const ptr[2] = {&accept, &next};
        for (int k = 0; k < 2; ++k) {
            if (a[6 + k] != Py_None) {        // also an empty one, whose pointer is null
                Py_INCREF(a[6 + k]);
                outputs[k] = a[6 + k];
            } else {
                fresh[k] = at::empty({n}, l->options().requires_grad(false));
                *ptr[k] = fresh[k].data_ptr();
            }
        }
        stream = current_stream(device);
        return true;
    }
    // (accept_len, next_token), or the status of a call that failed.
    PyObject* result(asd_status st) {
        if (st != ASD_OK) return PyLong_FromLong(st);
        for (int k = 0; k < 2; ++k)
            if (!outputs[k] && !(outputs[k] = THPVariable_Wrap(std::move(fresh[k])))) return nullptr;
        return PyTuple_Pack(2, outputs[0], outputs[1]);
    }
    ~Shared() {
        Py_XDECREF(outputs[0]);
        Py_XDECREF(outputs[1]);
    }
};

PyObject* done(asd_status st) {
    if (st != ASD_OK) return PyLong_FromLong(st);
    Py_RETURN_TRUE;
}

template <typename F>
F entry(PyObject* address) {
    return reinterpret_cast<F>(PyLong_AsVoidPtr(address));
}

// Runs a library call without the interpreter lock.
template <typename Call>
asd_status unlocked(Call&& call) {
    asd_status st;
    Py_BEGIN_ALLOW_THREADS;
    st = call();
    Py_END_ALLOW_THREADS;
    return st;
}

// Logits [rows, V] in f32 or bf16: type code, sizes and pointer.
struct Logits {
    asd_dtype dtype;
    int64_t rows, vocab;
    void* ptr;
    bool take(PyObject* o, int device) {
        const at::Tensor* t = dense(o, ScalarType::BFloat16, device);
        dtype = ASD_BF16;
        if (!t) {
            t = dense(o, ScalarType::Float, device);
            dtype = ASD_F32;
        }
        if (!t || t->dim() != 2) return false;
        rows = t->size(0);
        vocab = t->size(1);
        ptr = t->data_ptr();
        return true;
    }
};

// verify(entry, logits, shared...): asd_verify and asd_verify_static
PyObject* verify(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 2 + kShared) Py_RETURN_NONE;
    const int device = current_device(a[1]);
    Logits z;
    Shared s;
    if (device < 0 || !z.take(a[1], device) || !s.take(a + 2, z.rows, device)) Py_RETURN_NONE;
    const auto f = entry<decltype(&asd_verify)>(a[0]);
    return s.result(unlocked([&] {
        return f(z.ptr, z.dtype, z.vocab, s.n, s.rows, (const int32_t*)s.draft,
                 (const int32_t*)s.lens, (const int64_t*)s.offsets, (const float*)s.tau,
                 (const int32_t*)s.cap, (asd_budget*)s.budget, (int32_t*)s.accept,
                 (int32_t*)s.next, (int32_t*)s.argmax, (float*)s.regret, s.stream);
    }));
    END_HANDLE_TH_ERRORS
}

// verify_ex(entry, logits, flags, shared...): the library's workspace
PyObject* verify_ex(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 3 + kShared || !PyLong_CheckExact(a[2])) Py_RETURN_NONE;
    const long flags = PyLong_AsLong(a[2]);
    if (flags < 0 || flags > (long)INT32_MAX) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const int device = current_device(a[1]);
    Logits z;
    Shared s;
    if (device < 0 || !z.take(a[1], device) || !s.take(a + 3, z.rows, device)) Py_RETURN_NONE;
    const auto f = entry<decltype(&asd_verify_ex)>(a[0]);
    return s.result(unlocked([&] {
        return f(z.ptr, z.dtype, z.vocab, s.n, s.rows, (const int32_t*)s.draft,
                 (const int32_t*)s.lens, (const int64_t*)s.offsets, (const float*)s.tau,
                 (const int32_t*)s.cap, (asd_budget*)s.budget, (int32_t*)s.accept,
                 (int32_t*)s.next, (int32_t*)s.argmax, (float*)s.regret, (uint32_t)flags, s.stream,
                 nullptr, 0);
    }));
    END_HANDLE_TH_ERRORS
}

// verify_commit(entry, logits, tokens, seq_len, committed, shared...)
PyObject* verify_commit(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 5 + kShared) Py_RETURN_NONE;
    const int device = current_device(a[1]);
    Logits z;
    Shared s;
    if (device < 0 || !z.take(a[1], device)) Py_RETURN_NONE;
    const at::Tensor* tokens = dense(a[2], ScalarType::Int, device);
    const at::Tensor* lens = dense(a[6], ScalarType::Int, device);
    void *seq_len, *committed;
    if (!tokens || tokens->dim() != 2 || !lens || lens->dim() != 1 ||
        tokens->size(0) != lens->size(0) ||
        !vec(a[3], ScalarType::Long, lens->size(0), device, &seq_len) ||
        !vec(a[4], ScalarType::Int, lens->size(0), device, &committed, true) ||
        !s.take(a + 5, z.rows, device))
        Py_RETURN_NONE;
    void* const t = tokens->data_ptr();
    const int64_t capacity = tokens->size(1);
    const auto f = entry<decltype(&asd_verify_commit)>(a[0]);
    return s.result(unlocked([&] {
        return f(z.ptr, z.dtype, z.vocab, s.n, s.rows, (const int32_t*)s.draft,
                 (const int32_t*)s.lens, (const int64_t*)s.offsets, (const float*)s.tau,
                 (const int32_t*)s.cap, (asd_budget*)s.budget, (int32_t*)s.accept,
                 (int32_t*)s.next, (int32_t*)s.argmax, (float*)s.regret, (int32_t*)t, capacity,
                 (int64_t*)seq_len, (int32_t*)committed, s.stream, nullptr, 0);
    }));
    END_HANDLE_TH_ERRORS
}

bool integer(PyObject* o, int64_t* out) {
    if (!PyLong_CheckExact(o)) return false;
    *out = PyLong_AsLongLong(o);
    if (*out == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

// verify_partials(entry, partials, shard_vocab, vocab, shared...)
PyObject* verify_partials(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 4 + kShared) Py_RETURN_NONE;
    const int device = current_device(a[1]);
    int64_t width, vocab;
    const at::Tensor* p = device < 0 ? nullptr : dense(a[1], ScalarType::Int, device);
    Shared s;
    if (!p || p->dim() != 3 || p->size(2) != 4 || p->size(0) > INT32_MAX || !integer(a[2], &width) ||
        !integer(a[3], &vocab) || !s.take(a + 4, p->size(1), device))
        Py_RETURN_NONE;
    const void* const ptr = p->data_ptr();
    const int32_t shards = (int32_t)p->size(0);
    const auto f = entry<decltype(&asd_verify_partials)>(a[0]);
    return s.result(unlocked([&] {
        return f((const asd_row_partial*)ptr, shards, width, vocab, s.n, s.rows,
                 (const int32_t*)s.draft, (const int32_t*)s.lens, (const int64_t*)s.offsets,
                 (const float*)s.tau, (const int32_t*)s.cap, (asd_budget*)s.budget,
                 (int32_t*)s.accept, (int32_t*)s.next, (int32_t*)s.argmax, (float*)s.regret,
                 s.stream);
    }));
    END_HANDLE_TH_ERRORS
}

// lmhead_verify(entry, hidden, weight, shared...)
PyObject* lmhead_verify(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 3 + kShared) Py_RETURN_NONE;
    const int device = current_device(a[1]);
    if (device < 0) Py_RETURN_NONE;
    const at::Tensor* h = dense(a[1], ScalarType::BFloat16, device);
    const at::Tensor* w = dense(a[2], ScalarType::BFloat16, device);
    Shared s;
    if (!h || !w || h->dim() != 2 || w->dim() != 2 || h->size(1) != w->size(1) ||
        !s.take(a + 3, h->size(0), device))
        Py_RETURN_NONE;
    const void *hp = h->data_ptr(), *wp = w->data_ptr();
    const int64_t d = h->size(1), vocab = w->size(0);
    const auto f = entry<decltype(&asd_lmhead_verify)>(a[0]);
    return s.result(unlocked([&] {
        return f(hp, wp, d, vocab, s.n, s.rows, (const int32_t*)s.draft, (const int32_t*)s.lens,
                 (const int64_t*)s.offsets, (const float*)s.tau, (const int32_t*)s.cap,
                 (asd_budget*)s.budget, (int32_t*)s.accept, (int32_t*)s.next, (int32_t*)s.argmax,
                 (float*)s.regret, s.stream);
    }));
    END_HANDLE_TH_ERRORS
}

// shard_argmax(entry, shard_logits, vocab_offset, vocab, draft, partials)
PyObject* shard_argmax(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 6) Py_RETURN_NONE;
    const int device = current_device(a[1]);
    Logits z;
    int64_t offset, vocab;
    void* draft;
    if (device < 0 || !z.take(a[1], device) || !integer(a[2], &offset) || !integer(a[3], &vocab) ||
        !vec(a[4], ScalarType::Int, z.rows, device, &draft))
        Py_RETURN_NONE;
    const at::Tensor* p = dense(a[5], ScalarType::Int, device);
    if (!p || p->dim() != 2 || p->size(0) != z.rows || p->size(1) != 4) Py_RETURN_NONE;
    void *out = p->data_ptr(), *stream = current_stream(device);
    const auto f = entry<decltype(&asd_shard_argmax)>(a[0]);
    return done(unlocked([&] {
        return f(z.ptr, z.dtype, z.vocab, offset, vocab, z.rows, (const int32_t*)draft,
                 (asd_row_partial*)out, stream);
    }));
    END_HANDLE_TH_ERRORS
}

// opportunity(entry, draft, argmax, regret, vocab, lens, taus, ps, counts,
// mismatches, offsets)
PyObject* opportunity(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 11) Py_RETURN_NONE;
    const int device = current_device(a[1]);
    if (device < 0) Py_RETURN_NONE;
    const at::Tensor* x = dense(a[1], ScalarType::Int, device);
    const at::Tensor* lens = dense(a[5], ScalarType::Int, device);
    const at::Tensor* taus = dense(a[6], ScalarType::Float, device);
    const at::Tensor* ps = dense(a[7], ScalarType::Int, device);
    const at::Tensor* counts = dense(a[8], ScalarType::Long, device);
    int64_t vocab;
    void *argmax, *regret, *mismatches, *offsets;
    if (!x || x->dim() != 1 || !lens || lens->dim() != 1 || lens->size(0) > INT32_MAX || !taus ||
        taus->dim() != 1 || taus->size(0) > INT32_MAX || !ps || ps->dim() != 1 ||
        ps->size(0) > INT32_MAX || !counts || counts->dim() != 2 ||
        counts->size(0) != taus->size(0) || counts->size(1) != ps->size(0) ||
        !integer(a[4], &vocab) || !vec(a[2], ScalarType::Int, x->size(0), device, &argmax) ||
        !vec(a[3], ScalarType::Float, x->size(0), device, &regret) ||
        !vec(a[9], ScalarType::Long, 1, device, &mismatches) ||
        !vec(a[10], ScalarType::Long, lens->size(0), device, &offsets, true))
        Py_RETURN_NONE;
    const int64_t rows = x->size(0);
    const int32_t n = (int32_t)lens->size(0), nt = (int32_t)taus->size(0), np = (int32_t)ps->size(0);
    void *xp = x->data_ptr(), *lp = lens->data_ptr(), *tp = taus->data_ptr(), *pp = ps->data_ptr();
    void *cp = counts->data_ptr(), *stream = current_stream(device);
    const auto f = entry<decltype(&asd_opportunity)>(a[0]);
    return done(unlocked([&] {
        return f((const int32_t*)xp, (const int32_t*)argmax, (const float*)regret, vocab, n, rows,
                 (const int32_t*)lp, (const int64_t*)offsets, (const float*)tp, nt,
                 (const int32_t*)pp, np, (uint64_t*)cp, (uint64_t*)mismatches, stream);
    }));
    END_HANDLE_TH_ERRORS
}

PyObject* source_hash(PyObject*, PyObject*) { return PyUnicode_FromString(ASD_BINDING_HASH); }

#define ASD_FAST(name) \
    {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ASD_FAST(verify),        ASD_FAST(verify_ex),
                         ASD_FAST(verify_commit), ASD_FAST(verify_partials),
                         ASD_FAST(lmhead_verify), ASD_FAST(shard_argmax),
                         ASD_FAST(opportunity),   {"source_hash", source_hash, METH_NOARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_asd_binding", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__asd_binding(void) { return PyModule_Create(&module); }
