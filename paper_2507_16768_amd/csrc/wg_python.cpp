// The Python side's per-step calls, as native code: what binding.py offers as methods checks its
// tensors, finds the current stream and calls the C ABI from here.  A decode step of a small batch
// is bound by the host, and the same checks written in Python over ctypes took 8 us of the 13 us a
// step took (B = 1); here the whole call is about the launches.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>

#include <cstring>
#include <exception>
#include <string>
#include <vector>

#include "../../include/wg.h"

namespace {

PyObject *g_error = nullptr;             // binding.WgError

// Raises; always returns false / nullptr so that callers can return it.
bool bad(PyObject *type, const std::string &msg) { PyErr_SetString(type, msg.c_str()); return false; }

PyObject *result(int rc) {
    if (rc == WG_OK) Py_RETURN_NONE;
    PyObject *e = PyObject_CallFunction(g_error, "iN", rc, PyUnicode_DecodeUTF8(wg_last_error(), (Py_ssize_t)std::strlen(wg_last_error()), "replace"));
    if (e) { PyErr_SetObject(g_error, e); Py_DECREF(e); }
    return nullptr;
}

bool count(Py_ssize_t n, Py_ssize_t want) { return n == want || bad(PyExc_TypeError, "wrong number of arguments"); }

bool tensor(PyObject *o, const at::Tensor **out, const char *name) {
    if (!THPVariable_Check(o)) return bad(PyExc_TypeError, std::string(name) + " must be a tensor");
    *out = &THPVariable_Unpack(o);
    return true;
}
// A contiguous device tensor of one type.
bool device(const at::Tensor &t, at::ScalarType dtype, const char *name) {
    if (!t.is_cuda() || !t.is_contiguous()) return bad(PyExc_ValueError, std::string(name) + " must be a contiguous device tensor");
    if (t.scalar_type() != dtype)
        return bad(PyExc_ValueError, std::string(name) + " must have dtype torch." + (dtype == at::kInt ? "int32" : dtype == at::kLong ? "int64" :
                                     dtype == at::kByte ? "uint8" : dtype == at::kFloat ? "float32" : "bfloat16"));
    return true;
}
bool shape2(const at::Tensor &t, int64_t a, int64_t b) { return t.dim() == 2 && t.size(0) == a && t.size(1) == b; }
bool shape1(const at::Tensor &t, int64_t a) { return t.dim() == 1 && t.size(0) == a; }

// None: torch's current stream; a torch stream; or an address.
bool stream_of(PyObject *o, void **out) {
    if (o == Py_None) { *out = c10::hip::getCurrentHIPStream().stream(); return true; }
    PyObject *s = PyObject_HasAttrString(o, "cuda_stream") ? PyObject_GetAttrString(o, "cuda_stream") : PyNumber_Long(o);
    if (!s) return false;
    *out = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    return !PyErr_Occurred();
}
bool handle_of(PyObject *o, wg_handle_t *out) {
    *out = static_cast<wg_handle_t>(PyLong_AsVoidPtr(o));
    return !PyErr_Occurred();
}

// The C call f() without the interpreter's lock.  f captures addresses and numbers, no tensors: what asks
// a tensor may throw (a tensor without storage, as vmap, functorch and fake modes hand them in) and may
// call back into Python, so it is done before, with the lock held.
template <typename F> int unlocked(F f) {
    struct Release {
        PyThreadState *state = PyEval_SaveThread();
        ~Release() { PyEval_RestoreThread(state); }
    } released;
    return f();
}

// A method of the module: C++ exceptions become Python's, as torch's own calls translate them.
using Method = PyObject *(PyObject *, PyObject *const *, Py_ssize_t);
template <Method *f> PyObject *guarded(PyObject *self, PyObject *const *a, Py_ssize_t n) {
    try {
        return f(self, a, n);
    } catch (...) {
        torch::translate_exception_to_python(std::current_exception());
        return nullptr;
    }
}

bool states_ok(const at::Tensor &t) { return t.dim() == 2 && t.size(1) == 2; }
wg_state_t *states_ptr(const at::Tensor &t) { return static_cast<wg_state_t *>(t.data_ptr()); }
uint32_t *words(const at::Tensor &t) { return static_cast<uint32_t *>(t.data_ptr()); }
int32_t *ints(const at::Tensor &t) { return static_cast<int32_t *>(t.data_ptr()); }
uint32_t rows(const at::Tensor &t) { return (uint32_t)t.size(0); }

// A [B, V] float32 or bfloat16 device tensor with unit inner stride.
bool logits_ok(const at::Tensor &t, wg_dtype_t *dt, const char *what) {
    if (t.dim() != 2 || !t.is_cuda() || t.stride(1) != 1) return bad(PyExc_ValueError, what);
    if (t.scalar_type() == at::kFloat) *dt = WG_F32;
    else if (t.scalar_type() == at::kBFloat16) *dt = WG_BF16;
    else return bad(PyExc_ValueError, "logits must be float32 or bfloat16");
    return true;
}

// fill_masks(handle, W, states, bitmask, stream)
PyObject *fill_masks(PyObject *, PyObject *const *a, Py_ssize_t n) {
    wg_handle_t h; const at::Tensor *st, *bm; void *s;
    if (!count(n, 5) || !handle_of(a[0], &h) || !tensor(a[2], &st, "states") || !tensor(a[3], &bm, "bitmask")) return nullptr;
    const int64_t W = PyLong_AsLongLong(a[1]);
    if (!states_ok(*st) || !shape2(*bm, st->size(0), W)) { bad(PyExc_ValueError, "states must be [B, 2] and bitmask [B, W]"); return nullptr; }
    if (!device(*st, at::kInt, "states") || !device(*bm, at::kInt, "bitmask") || !stream_of(a[4], &s)) return nullptr;
    return result(unlocked([=, states = states_ptr(*st), B = rows(*st), mask = words(*bm)] { return wg_fill_masks(h, states, B, mask, s); }));
}

// advance(handle, states, tokens, stream)
PyObject *advance(PyObject *, PyObject *const *a, Py_ssize_t n) {
    wg_handle_t h; const at::Tensor *st, *tk; void *s;
    if (!count(n, 4) || !handle_of(a[0], &h) || !tensor(a[1], &st, "states") || !tensor(a[2], &tk, "tokens")) return nullptr;
    if (!states_ok(*st) || !shape1(*tk, st->size(0))) { bad(PyExc_ValueError, "states must be [B, 2] and tokens [B]"); return nullptr; }
    if (!device(*st, at::kInt, "states") || !device(*tk, at::kInt, "tokens") || !stream_of(a[3], &s)) return nullptr;
    return result(unlocked([=, states = states_ptr(*st), tokens = ints(*tk), B = rows(*st)] { return wg_advance(h, states, tokens, B, s); }));
}

// advance_fill_masks(handle, W, states, tokens, bitmask, stream)
PyObject *advance_fill_masks(PyObject *, PyObject *const *a, Py_ssize_t n) {
    wg_handle_t h; const at::Tensor *st, *tk, *bm; void *s;
    if (!count(n, 6) || !handle_of(a[0], &h) || !tensor(a[2], &st, "states") || !tensor(a[3], &tk, "tokens") || !tensor(a[4], &bm, "bitmask")) return nullptr;
    const int64_t W = PyLong_AsLongLong(a[1]);
    if (!states_ok(*st) || !shape1(*tk, st->size(0)) || !shape2(*bm, st->size(0), W)) {
        bad(PyExc_ValueError, "states must be [B, 2], tokens [B] and bitmask [B, W]");
        return nullptr;
    }
    if (!device(*st, at::kInt, "states") || !device(*tk, at::kInt, "tokens") || !device(*bm, at::kInt, "bitmask") || !stream_of(a[5], &s)) return nullptr;
    return result(unlocked([=, states = states_ptr(*st), tokens = ints(*tk), B = rows(*st), mask = words(*bm)] {
        return wg_advance_fill_masks(h, states, tokens, B, mask, s);
    }));
}

// decode_step(handle, W, V, states, tokens or None, bitmask, logits, stream)
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
    wg_handle_t h; const at::Tensor *st, *tk = nullptr, *bm, *lg; void *s; wg_dtype_t dt;
    if (!count(n, 8) || !handle_of(a[0], &h) || !tensor(a[3], &st, "states") || (a[4] != Py_None && !tensor(a[4], &tk, "tokens")) ||
        !tensor(a[5], &bm, "bitmask") || !tensor(a[6], &lg, "logits")) return nullptr;
    const int64_t W = PyLong_AsLongLong(a[1]), V = PyLong_AsLongLong(a[2]);
    if (!states_ok(*st) || !shape2(*bm, st->size(0), W)) { bad(PyExc_ValueError, "states must be [B, 2] and bitmask [B, W]"); return nullptr; }
    if (tk && !shape1(*tk, st->size(0))) { bad(PyExc_ValueError, "tokens must be [B]"); return nullptr; }
    if (!logits_ok(*lg, &dt, "logits must be a [B, V] device tensor with unit inner stride")) return nullptr;
    if (lg->size(0) != st->size(0)) { bad(PyExc_ValueError, "logits must be a [B, V] device tensor with unit inner stride"); return nullptr; }
    if (lg->size(1) != V) { bad(PyExc_ValueError, "logits must have the vocabulary's width"); return nullptr; }
    if (!device(*st, at::kInt, "states") || (tk && !device(*tk, at::kInt, "tokens")) || !device(*bm, at::kInt, "bitmask") || !stream_of(a[7], &s)) return nullptr;
    return result(unlocked([=, states = states_ptr(*st), tokens = tk ? ints(*tk) : nullptr, B = rows(*st), mask = words(*bm), logits = lg->data_ptr(),
                            stride = lg->stride(0)] { return wg_decode_step(h, states, tokens, B, mask, logits, dt, stride, s); }));
}

// forced_bytes(handle, states, out_bytes, out_lens, end_states or None, stream)
PyObject *forced_bytes(PyObject *, PyObject *const *a, Py_ssize_t n) {
    wg_handle_t h; const at::Tensor *st, *ob, *ol, *es = nullptr; void *s;
    if (!count(n, 6) || !handle_of(a[0], &h) || !tensor(a[1], &st, "states") || !tensor(a[2], &ob, "out_bytes") || !tensor(a[3], &ol, "out_lens") ||
        (a[4] != Py_None && !tensor(a[4], &es, "end_states"))) return nullptr;
    if (!states_ok(*st) || ob->dim() != 2 || ob->size(0) != st->size(0) || !shape1(*ol, st->size(0))) {
        bad(PyExc_ValueError, "states must be [B, 2], out_bytes [B, cap] and out_lens [B]");
        return nullptr;
    }
    if (es && !shape2(*es, st->size(0), 2)) { bad(PyExc_ValueError, "end_states must be [B, 2]"); return nullptr; }
    if (!device(*st, at::kInt, "states") || !device(*ob, at::kByte, "out_bytes") || !device(*ol, at::kInt, "out_lens") ||
        (es && !device(*es, at::kInt, "end_states")) || !stream_of(a[5], &s)) return nullptr;
    return result(unlocked([=, states = states_ptr(*st), B = rows(*st), cap = (uint32_t)ob->size(1), bytes = static_cast<uint8_t *>(ob->data_ptr()),
                            lens = words(*ol), ends = es ? states_ptr(*es) : nullptr] { return wg_forced_bytes(h, states, B, cap, bytes, lens, ends, s); }));
}

// cache_clear(handle, stream)
PyObject *cache_clear(PyObject *, PyObject *const *a, Py_ssize_t n) {
    wg_handle_t h; void *s;
    if (!count(n, 2) || !handle_of(a[0], &h) || !stream_of(a[1], &s)) return nullptr;
    return result(wg_cache_clear(h, s));
}

// What the sampling calls share: logits [B, V] and a bitmask [B, ceil(V / 32)].
bool masked(PyObject *lo, PyObject *bo, const at::Tensor **lg, const at::Tensor **bm, wg_dtype_t *dt) {
    if (!tensor(lo, lg, "logits") || !tensor(bo, bm, "bitmask") || !logits_ok(**lg, dt, "logits must be a 2-d device tensor with unit inner stride")) return false;
    return true;
}
bool mask_fits(const at::Tensor &lg, const at::Tensor &bm) { return shape2(bm, lg.size(0), (lg.size(1) + 31) / 32); }

// apply_mask(logits, bitmask, stream)
PyObject *apply_mask(PyObject *, PyObject *const *a, Py_ssize_t n) {
    const at::Tensor *lg, *bm; void *s; wg_dtype_t dt;
    if (!count(n, 3) || !masked(a[0], a[1], &lg, &bm, &dt)) return nullptr;
    if (!mask_fits(*lg, *bm)) { bad(PyExc_ValueError, "bitmask must be [B, ceil(V/32)]"); return nullptr; }
    if (!device(*bm, at::kInt, "bitmask") || !stream_of(a[2], &s)) return nullptr;
    return result(unlocked([=, logits = lg->data_ptr(), B = rows(*lg), V = (uint32_t)lg->size(1), stride = lg->stride(0), mask = words(*bm)] {
        return wg_apply_mask(logits, dt, B, V, stride, mask, s);
    }));
}

// masked_argmax(logits, bitmask, tokens, stream)
PyObject *masked_argmax(PyObject *, PyObject *const *a, Py_ssize_t n) {
    const at::Tensor *lg, *bm, *tk; void *s; wg_dtype_t dt;
    if (!count(n, 4) || !masked(a[0], a[1], &lg, &bm, &dt) || !tensor(a[2], &tk, "tokens")) return nullptr;
    if (!mask_fits(*lg, *bm) || !shape1(*tk, lg->size(0))) { bad(PyExc_ValueError, "bitmask must be [B, ceil(V/32)] and tokens [B]"); return nullptr; }
    if (!device(*bm, at::kInt, "bitmask") || !device(*tk, at::kInt, "tokens") || !stream_of(a[3], &s)) return nullptr;
    return result(unlocked([=, logits = lg->data_ptr(), B = rows(*lg), V = (uint32_t)lg->size(1), stride = lg->stride(0), mask = words(*bm), tokens = ints(*tk)] {
        return wg_masked_argmax(logits, dt, B, V, stride, mask, tokens, s);
    }));
}

// masked_topk(logits, bitmask, ids, values, workspace or None (the library's own), stream)
PyObject *masked_topk(PyObject *, PyObject *const *a, Py_ssize_t n) {
    const at::Tensor *lg, *bm, *id, *va, *ws = nullptr; void *s; wg_dtype_t dt;
    if (!count(n, 6) || !masked(a[0], a[1], &lg, &bm, &dt) || !tensor(a[2], &id, "ids") || !tensor(a[3], &va, "values") ||
        (a[4] != Py_None && !tensor(a[4], &ws, "workspace"))) return nullptr;
    if (id->dim() != 2 || id->size(0) != lg->size(0) || va->sizes() != id->sizes()) { bad(PyExc_ValueError, "ids and values must be [B, k]"); return nullptr; }
    if (!mask_fits(*lg, *bm)) { bad(PyExc_ValueError, "bitmask must be [B, ceil(V/32)]"); return nullptr; }
    if (!device(*bm, at::kInt, "bitmask") || !device(*id, at::kInt, "ids") || !device(*va, lg->scalar_type(), "values") ||
        (ws && !device(*ws, ws->scalar_type(), "workspace")) || !stream_of(a[5], &s)) return nullptr;
    const uint32_t B = rows(*lg), V = (uint32_t)lg->size(1), k = (uint32_t)id->size(1);
    const bool own = !ws;
    return result(unlocked([=, logits = lg->data_ptr(), stride = lg->stride(0), mask = words(*bm), ids = ints(*id), values = va->data_ptr(),
                            work = ws ? ws->data_ptr() : nullptr, bytes = ws ? (uint64_t)ws->numel() * ws->element_size() : 0u] {
        return own ? wg_masked_topk_static(logits, dt, B, V, stride, mask, k, ids, values, s)
                   : wg_masked_topk(logits, dt, B, V, stride, mask, k, ids, values, work, bytes, s);
    }));
}

// select_tokens(bitmask, V, draws, tokens, stream)
PyObject *select_tokens(PyObject *, PyObject *const *a, Py_ssize_t n) {
    const at::Tensor *bm, *dr, *tk; void *s;
    if (!count(n, 5) || !tensor(a[0], &bm, "bitmask") || !tensor(a[2], &dr, "draws") || !tensor(a[3], &tk, "tokens")) return nullptr;
    const int64_t V = PyLong_AsLongLong(a[1]);
    if (PyErr_Occurred() || !device(*bm, at::kInt, "bitmask") || !device(*dr, at::kLong, "draws") || !device(*tk, at::kInt, "tokens") || !stream_of(a[4], &s)) return nullptr;
    return result(unlocked([=, mask = words(*bm), B = bm->dim() ? rows(*bm) : 0u, draws = static_cast<const uint64_t *>(dr->data_ptr()), tokens = ints(*tk)] {
        return wg_select_tokens(mask, B, (uint32_t)V, draws, tokens, s);
    }));
}

// add_instances(handle, texts, args or None, starts address, its rows, stream): sequences of template texts and of
// argument mappings.  The C call reads the strings in place and without the lock, when other threads may
// change the caller's lists and dictionaries, and a conversion to bytes may run Python code that does:
// a reference is held to everything that is pointed into, and no container is walked after such code ran.
PyObject *add_instances(PyObject *, PyObject *const *a, Py_ssize_t n) {
    wg_handle_t h; void *s;
    if (!count(n, 6) || !handle_of(a[0], &h) || !stream_of(a[5], &s)) return nullptr;
    void *starts = PyLong_AsVoidPtr(a[3]);
    const Py_ssize_t room = PyLong_AsSsize_t(a[4]);
    if (PyErr_Occurred()) return nullptr;
    struct Refs {                                      // what has to live until the call is over
        std::vector<PyObject *> v;
        ~Refs() { for (PyObject *o : v) Py_DECREF(o); }
        PyObject *keep(PyObject *o) {                  // takes over a new reference
            if (o) try { v.push_back(o); } catch (...) { Py_DECREF(o); throw; }
            return o;
        }
    } refs;
    PyObject *texts = refs.keep(PySequence_Tuple(a[1]));
    if (!texts) return nullptr;
    const Py_ssize_t count_ = PyTuple_GET_SIZE(texts);
    if (count_ > room) { bad(PyExc_ValueError, "more templates than the result has rows"); return nullptr; }
    std::vector<const char *> c_texts((size_t)count_ + 1, nullptr);
    // o is held by the caller of this; what is made from it here is held by refs
    auto bytes_of = [&](PyObject *o, const char **p, uint64_t *len) {
        if (PyUnicode_Check(o)) { Py_ssize_t k; *p = PyUnicode_AsUTF8AndSize(o, &k); if (len) *len = (uint64_t)k; return *p != nullptr; }
        PyObject *b = o;
        if (!PyBytes_Check(o)) { b = refs.keep(PyObject_CallFunctionObjArgs((PyObject *)&PyBytes_Type, o, nullptr)); if (!b) return false; }
        *p = PyBytes_AS_STRING(b);
        if (len) *len = (uint64_t)PyBytes_GET_SIZE(b);
        return true;
    };
    for (Py_ssize_t i = 0; i < count_; i++)
        if (!bytes_of(PyTuple_GET_ITEM(texts, i), &c_texts[i], nullptr)) return nullptr;
    std::vector<wg_args_t> c_args;
    std::vector<const char *> names;
    std::vector<const uint8_t *> data;
    std::vector<uint64_t> lens;
    if (a[2] != Py_None) {
        PyObject *args = refs.keep(PySequence_Tuple(a[2]));
        if (!args) return nullptr;
        if (PyTuple_GET_SIZE(args) != count_) { bad(PyExc_ValueError, "one argument set per template is required"); return nullptr; }
        std::vector<size_t> first((size_t)count_ + 1, 0);
        std::vector<PyObject *> items;                 // names and values of one set, in turn
        for (Py_ssize_t i = 0; i < count_; i++) {
            PyObject *d = PyTuple_GET_ITEM(args, i), *key, *value;
            if (!PyDict_Check(d) && !(d = refs.keep(PyObject_CallFunctionObjArgs((PyObject *)&PyDict_Type, d, nullptr)))) return nullptr;
            items.clear();
            Py_ssize_t at = 0;
            while (PyDict_Next(d, &at, &key, &value)) {
                if (!PyUnicode_Check(key) || PyUnicode_Check(value)) { bad(PyExc_TypeError, "arguments map names to bytes"); return nullptr; }
                Py_INCREF(key); items.push_back(refs.keep(key));
                Py_INCREF(value); items.push_back(refs.keep(value));
            }
            for (size_t k = 0; k < items.size(); k += 2) {
                const char *p; uint64_t len;
                if (!bytes_of(items[k], &p, nullptr)) return nullptr;
                names.push_back(p);
                if (!bytes_of(items[k + 1], &p, &len)) return nullptr;
                data.push_back(reinterpret_cast<const uint8_t *>(p)); lens.push_back(len);
            }
            first[i + 1] = names.size();
        }
        names.push_back(nullptr); data.push_back(nullptr); lens.push_back(0);
        for (Py_ssize_t i = 0; i < count_; i++)
            c_args.push_back(wg_args_t{(uint32_t)(first[i + 1] - first[i]), &names[first[i]], &data[first[i]], &lens[first[i]]});
        c_args.push_back(wg_args_t{});
    }
    return result(unlocked([&] {
        return wg_add_instances(h, c_texts.data(), c_args.empty() ? nullptr : c_args.data(), (uint32_t)count_, static_cast<wg_state_t *>(starts), s);
    }));
}

PyObject *set_error(PyObject *, PyObject *cls) {
    Py_INCREF(cls);
    Py_XDECREF(g_error);
    g_error = cls;
    Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(guarded<name>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(fill_masks), FAST(advance), FAST(advance_fill_masks), FAST(decode_step), FAST(forced_bytes), FAST(cache_clear),
                         FAST(apply_mask), FAST(masked_argmax), FAST(masked_topk), FAST(select_tokens), FAST(add_instances),
                         {"set_error", set_error, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
