// The per-call work of the Python binding in native code: checks a call's tensors against
// its descriptor, takes their addresses and the current stream, and calls the C ABI.
//
// A codec call on a small message is over in a few microseconds on the device, so what the
// host does per call decides how fast a training loop can issue them.  The same checks in
// Python (some twenty attribute reads and four foreign calls for size formulas) took 7.0 us
// per encode call next to the launch's 2.9 us, and 3.3 us per job; here 0.3 and 0.2 us.
// Four calls on a 131072-element message: 33.7 -> 16.2 us.
//
// Every function returns the library's status, or None when the call is not of the
// ordinary form (a tensor of another type, size or place, a stream that is no torch
// stream, ...).  binding.py then takes its own path, which knows how to explain what is
// wrong; nothing is decided here that it would decide differently.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <vector>

#include "aqsgd.h"

namespace {

// The library's entry points, by address: binding.py loads the library (whichever build
// AQSGD_LIB names) and hands them over.
struct Api {
    decltype(&aqsgd_codes_bytes) codes_bytes;
    decltype(&aqsgd_scales_count) scales_count;
    decltype(&aqsgd_lowbit_row_bytes) lowbit_row_bytes;
    decltype(&aqsgd_topk_bitmap_bytes) topk_bitmap_bytes;
    decltype(&aqsgd_topk_codes_bytes) topk_codes_bytes;
    decltype(&aqsgd_encode) encode;
    decltype(&aqsgd_decode) decode;
    decltype(&aqsgd_grad_quant) grad_quant;
    decltype(&aqsgd_grad_dequant) grad_dequant;
    decltype(&aqsgd_seed) seed;
    decltype(&aqsgd_encode_seen) encode_seen;
    decltype(&aqsgd_decode_seen) decode_seen;
    decltype(&aqsgd_encode_lowbit) encode_lowbit;
    decltype(&aqsgd_decode_lowbit) decode_lowbit;
    decltype(&aqsgd_grad_topk_quant) grad_topk_quant;
    decltype(&aqsgd_grad_topk_dequant) grad_topk_dequant;
    decltype(&aqsgd_run_jobs) run_jobs;
};
Api g_api;
PyTypeObject* g_desc_type = nullptr;      // the binding's ctypes mirrors of aqsgd_desc and aqsgd_job
PyTypeObject* g_job_type = nullptr;

// The memory of a ctypes structure of exactly this type, while the view lives.
class View {
public:
    View(PyObject* o, PyTypeObject* type, size_t bytes) {
        if (Py_TYPE(o) != type) return;
        if (PyObject_GetBuffer(o, &view_, PyBUF_SIMPLE) != 0) {
            PyErr_Clear();
            return;
        }
        held_ = true;
        ok_ = static_cast<size_t>(view_.len) == bytes;
    }
    ~View() {
        if (held_) PyBuffer_Release(&view_);
    }
    View(const View&) = delete;
    View& operator=(const View&) = delete;
    explicit operator bool() const { return ok_; }
    template <typename T> T* as() const { return static_cast<T*>(view_.buf); }

private:
    Py_buffer view_;
    bool held_ = false, ok_ = false;
};

c10::ScalarType element_type(const aqsgd_desc& d) {
    switch (d.dtype) {
    case AQSGD_F32: return c10::ScalarType::Float;
    case AQSGD_F16: return c10::ScalarType::Half;
    default:        return c10::ScalarType::BFloat16;
    }
}

// One call: its descriptor (copied: the sizes must be those that are checked) and the
// verdict over the tensors seen so far.
struct Call {
    aqsgd_desc d = {};
    int64_t n = 0;             // elements of a [batch, n_per] tensor
    bool ok = false;

    explicit Call(PyObject* desc) {
        View v(desc, g_desc_type, sizeof(aqsgd_desc));
        if (!v) return;
        std::memcpy(&d, v.as<aqsgd_desc>(), sizeof d);
        if (d.dtype != AQSGD_F32 && d.dtype != AQSGD_F16 && d.dtype != AQSGD_BF16) return;
        if (__builtin_mul_overflow(d.batch, d.n_per, &n)) return;
        ok = true;
    }

    void* tensor(PyObject* o, c10::ScalarType type, int64_t numel, bool exact) {
        if (!ok || !THPVariable_CheckExact(o)) { ok = false; return nullptr; }
        const at::Tensor& t = THPVariable_Unpack(o);
        ok = t.is_cuda() && t.scalar_type() == type && (exact ? t.numel() == numel : t.numel() >= numel) &&
             t.is_contiguous();
        return ok ? t.data_ptr() : nullptr;
    }
    void* row(PyObject* o) { return tensor(o, element_type(d), n, true); }
    void* ids(PyObject* o) { return tensor(o, c10::ScalarType::Long, d.batch, true); }
    void* m_buf(PyObject* o) {
        int64_t rows;
        if (__builtin_mul_overflow(d.n_samples, d.n_per, &rows)) ok = false;
        return ok ? tensor(o, element_type(d), rows, true) : nullptr;
    }
    void* bytes(PyObject* o, size_t least) { return tensor(o, c10::ScalarType::Byte, static_cast<int64_t>(least), false); }
    void* codes(PyObject* o) { return bytes(o, g_api.codes_bytes(&d)); }
    float* scales(PyObject* o) {
        return static_cast<float*>(tensor(o, c10::ScalarType::Float, static_cast<int64_t>(g_api.scales_count(&d)), false));
    }
    int32_t* words(PyObject* o, int64_t count) {
        return static_cast<int32_t*>(tensor(o, c10::ScalarType::Int, count, true));
    }
    int64_t number(PyObject* o) {
        if (!ok || !PyLong_CheckExact(o)) { ok = false; return 0; }
        int over = 0;
        const long long v = PyLong_AsLongLongAndOverflow(o, &over);
        if (over) ok = false;
        return v;
    }
    int32_t int32(PyObject* o) {
        const int64_t v = number(o);
        if (v != static_cast<int32_t>(v)) ok = false;
        return static_cast<int32_t>(v);
    }
    // None: the current stream of the current device; else a torch stream's handle
    void* stream(PyObject* o) {
        if (!ok) return nullptr;
        if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
        PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
        if (!h) { PyErr_Clear(); ok = false; return nullptr; }
        void* s = PyLong_Check(h) ? PyLong_AsVoidPtr(h) : nullptr;
        if (!PyLong_Check(h) || PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        Py_DECREF(h);
        return s;
    }
};

template <typename F>
PyObject* launch(const Call& c, F&& f) {
    if (!c.ok) Py_RETURN_NONE;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

// Argument counts are fixed by binding.py; a torch exception (a tensor without storage,
// say) means that the call is not of the ordinary form.
#define AQSGD_ENTRY(name, count, ...)                                             \
    PyObject* name(PyObject*, PyObject* const* p, Py_ssize_t np) {                \
        if (np != (count)) Py_RETURN_NONE;                                        \
        try __VA_ARGS__ catch (const std::exception&) { Py_RETURN_NONE; }         \
    }

using u8 = uint8_t;

AQSGD_ENTRY(py_encode, 7, {
    Call c(p[0]);
    void* act = c.row(p[1]); auto* ids = static_cast<int64_t*>(c.ids(p[2])); void* m = c.m_buf(p[3]);
    auto* codes = static_cast<u8*>(c.codes(p[4])); float* scales = c.scales(p[5]); void* s = c.stream(p[6]);
    return launch(c, [&] { return g_api.encode(&c.d, act, ids, m, codes, scales, s); });
})

AQSGD_ENTRY(py_decode, 7, {
    Call c(p[0]);
    auto* codes = static_cast<u8*>(c.codes(p[1])); float* scales = c.scales(p[2]);
    auto* ids = static_cast<int64_t*>(c.ids(p[3])); void* m = c.m_buf(p[4]); void* out = c.row(p[5]);
    void* s = c.stream(p[6]);
    return launch(c, [&] { return g_api.decode(&c.d, codes, scales, ids, m, out, s); });
})

AQSGD_ENTRY(py_grad_quant, 5, {
    Call c(p[0]);
    void* grad = c.row(p[1]); auto* codes = static_cast<u8*>(c.codes(p[2])); float* scales = c.scales(p[3]);
    void* s = c.stream(p[4]);
    return launch(c, [&] { return g_api.grad_quant(&c.d, grad, codes, scales, s); });
})

AQSGD_ENTRY(py_grad_dequant, 5, {
    Call c(p[0]);
    auto* codes = static_cast<u8*>(c.codes(p[1])); float* scales = c.scales(p[2]); void* out = c.row(p[3]);
    void* s = c.stream(p[4]);
    return launch(c, [&] { return g_api.grad_dequant(&c.d, codes, scales, out, s); });
})

AQSGD_ENTRY(py_seed, 5, {
    Call c(p[0]);
    void* act = c.row(p[1]); auto* ids = static_cast<int64_t*>(c.ids(p[2])); void* m = c.m_buf(p[3]);
    void* s = c.stream(p[4]);
    return launch(c, [&] { return g_api.seed(&c.d, act, ids, m, s); });
})

AQSGD_ENTRY(py_encode_seen, 10, {
    Call c(p[0]);
    void* act = c.row(p[1]); auto* ids = static_cast<int64_t*>(c.ids(p[2])); void* m = c.m_buf(p[3]);
    int32_t* seen = c.words(p[4], c.d.n_samples); const uint32_t stamp = static_cast<uint32_t>(c.number(p[5]));
    int32_t* first = c.words(p[6], c.d.batch);
    auto* codes = static_cast<u8*>(c.codes(p[7])); float* scales = c.scales(p[8]); void* s = c.stream(p[9]);
    return launch(c, [&] {
        return g_api.encode_seen(&c.d, act, ids, m, reinterpret_cast<uint32_t*>(seen), stamp, first, codes, scales, s);
    });
})

AQSGD_ENTRY(py_decode_seen, 10, {
    Call c(p[0]);
    auto* codes = static_cast<u8*>(c.codes(p[1])); float* scales = c.scales(p[2]); void* full = c.row(p[3]);
    auto* ids = static_cast<int64_t*>(c.ids(p[4])); void* m = c.m_buf(p[5]);
    int32_t* seen = c.words(p[6], c.d.n_samples); const uint32_t stamp = static_cast<uint32_t>(c.number(p[7]));
    void* out = c.row(p[8]); void* s = c.stream(p[9]);
    return launch(c, [&] {
        return g_api.decode_seen(&c.d, codes, scales, full, ids, m, reinterpret_cast<uint32_t*>(seen), stamp, out, s);
    });
})

// z-bit storage of the previous messages: levels and scales of every sample
struct LowbitStore {
    u8* codes = nullptr;
    float* scales = nullptr;
    LowbitStore(Call& c, int32_t z, PyObject* m_codes, PyObject* m_scales) {
        const size_t row = c.ok ? g_api.lowbit_row_bytes(&c.d, z) : 0;
        if (row == 0) { c.ok = false; return; }          // binding.py lets the library name the fault
        codes = static_cast<u8*>(c.tensor(m_codes, c10::ScalarType::Byte, c.d.n_samples * static_cast<int64_t>(row), true));
        scales = static_cast<float*>(c.tensor(m_scales, c10::ScalarType::Float, c.d.n_samples * (c.d.n_per / c.d.group), true));
    }
};

AQSGD_ENTRY(py_encode_lowbit, 9, {
    Call c(p[0]);
    const int32_t z = c.int32(p[1]);
    void* act = c.row(p[2]); auto* ids = static_cast<int64_t*>(c.ids(p[3]));
    const LowbitStore m(c, z, p[4], p[5]);
    auto* codes = static_cast<u8*>(c.codes(p[6])); float* scales = c.scales(p[7]); void* s = c.stream(p[8]);
    return launch(c, [&] { return g_api.encode_lowbit(&c.d, z, act, ids, m.codes, m.scales, codes, scales, s); });
})

AQSGD_ENTRY(py_decode_lowbit, 9, {
    Call c(p[0]);
    const int32_t z = c.int32(p[1]);
    auto* codes = static_cast<u8*>(c.codes(p[2])); float* scales = c.scales(p[3]);
    auto* ids = static_cast<int64_t*>(c.ids(p[4]));
    const LowbitStore m(c, z, p[5], p[6]);
    void* out = c.row(p[7]); void* s = c.stream(p[8]);
    return launch(c, [&] { return g_api.decode_lowbit(&c.d, z, codes, scales, ids, m.codes, m.scales, out, s); });
})

struct TopkMessage {
    u8 *bitmap = nullptr, *codes = nullptr;
    float* scales = nullptr;
    TopkMessage(Call& c, int32_t keep, PyObject* b, PyObject* q, PyObject* s) {
        const size_t nb = c.ok ? g_api.topk_bitmap_bytes(&c.d) : 0;
        const size_t nc = nb ? g_api.topk_codes_bytes(&c.d, keep) : 0;
        if (nc == 0) { c.ok = false; return; }           // binding.py lets the library name the fault
        bitmap = static_cast<u8*>(c.bytes(b, nb));
        codes = static_cast<u8*>(c.bytes(q, nc));
        scales = c.scales(s);
    }
};

AQSGD_ENTRY(py_grad_topk_quant, 7, {
    Call c(p[0]);
    const int32_t keep = c.int32(p[1]);
    void* grad = c.row(p[2]);
    const TopkMessage m(c, keep, p[3], p[4], p[5]);
    void* s = c.stream(p[6]);
    return launch(c, [&] { return g_api.grad_topk_quant(&c.d, keep, grad, m.bitmap, m.codes, m.scales, s); });
})

AQSGD_ENTRY(py_grad_topk_dequant, 7, {
    Call c(p[0]);
    const int32_t keep = c.int32(p[1]);
    const TopkMessage m(c, keep, p[2], p[3], p[4]);
    void* out = c.row(p[5]); void* s = c.stream(p[6]);
    return launch(c, [&] { return g_api.grad_topk_dequant(&c.d, keep, m.bitmap, m.codes, m.scales, out, s); });
})

// ---- jobs -------------------------------------------------------------------------------
PyObject* new_job(const Call& c, const aqsgd_job& j) {
    if (!c.ok) Py_RETURN_NONE;
    PyObject* o = PyObject_CallNoArgs(reinterpret_cast<PyObject*>(g_job_type));
    if (!o) return nullptr;
    View v(o, g_job_type, sizeof(aqsgd_job));
    if (!v) { Py_DECREF(o); Py_RETURN_NONE; }
    std::memcpy(v.as<aqsgd_job>(), &j, sizeof j);
    return o;
}

aqsgd_job blank_job(const Call& c, aqsgd_job_kind kind) {
    aqsgd_job j;
    std::memset(&j, 0, sizeof j);
    j.kind = kind;
    if (c.ok) j.desc = c.d;
    return j;
}

AQSGD_ENTRY(py_encode_job, 6, {
    Call c(p[0]);
    aqsgd_job j = blank_job(c, AQSGD_JOB_ENCODE);
    j.src = c.row(p[1]); j.sample_ids = static_cast<int64_t*>(c.ids(p[2])); j.m_buf = c.m_buf(p[3]);
    j.codes = static_cast<u8*>(c.codes(p[4])); j.scales = c.scales(p[5]);
    return new_job(c, j);
})

AQSGD_ENTRY(py_decode_job, 6, {
    Call c(p[0]);
    aqsgd_job j = blank_job(c, AQSGD_JOB_DECODE);
    j.codes = static_cast<u8*>(c.codes(p[1])); j.scales = c.scales(p[2]);
    j.sample_ids = static_cast<int64_t*>(c.ids(p[3])); j.m_buf = c.m_buf(p[4]); j.out = c.row(p[5]);
    return new_job(c, j);
})

AQSGD_ENTRY(py_grad_quant_job, 4, {
    Call c(p[0]);
    aqsgd_job j = blank_job(c, AQSGD_JOB_GRAD_QUANT);
    j.src = c.row(p[1]); j.codes = static_cast<u8*>(c.codes(p[2])); j.scales = c.scales(p[3]);
    return new_job(c, j);
})

AQSGD_ENTRY(py_grad_dequant_job, 4, {
    Call c(p[0]);
    aqsgd_job j = blank_job(c, AQSGD_JOB_GRAD_DEQUANT);
    j.codes = static_cast<u8*>(c.codes(p[1])); j.scales = c.scales(p[2]); j.out = c.row(p[3]);
    return new_job(c, j);
})

AQSGD_ENTRY(py_run_jobs, 2, {
    const bool list = PyList_CheckExact(p[0]);
    if (!list && !PyTuple_CheckExact(p[0])) Py_RETURN_NONE;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(p[0]);
    if (n > 4096) Py_RETURN_NONE;
    std::vector<aqsgd_job> jobs(static_cast<size_t>(n));
    for (Py_ssize_t k = 0; k < n; ++k) {
        View v(PySequence_Fast_GET_ITEM(p[0], k), g_job_type, sizeof(aqsgd_job));
        if (!v) Py_RETURN_NONE;
        std::memcpy(&jobs[static_cast<size_t>(k)], v.as<aqsgd_job>(), sizeof(aqsgd_job));
    }
    struct { bool ok = true; } c;
    void* s = nullptr;
    if (p[1] == Py_None) {
        s = c10::hip::getCurrentHIPStream().stream();
    } else {
        PyObject* h = PyObject_GetAttrString(p[1], "cuda_stream");
        if (!h) { PyErr_Clear(); Py_RETURN_NONE; }
        c.ok = PyLong_Check(h);
        if (c.ok) s = PyLong_AsVoidPtr(h);
        Py_DECREF(h);
        if (!c.ok || PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    }
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = g_api.run_jobs(jobs.data(), static_cast<int32_t>(n), s);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
})

// setup(Desc, Job, {name: address}): called once by binding.py after it has loaded the library.
PyObject* py_setup(PyObject*, PyObject* const* p, Py_ssize_t np) {
    if (np != 3 || !PyType_Check(p[0]) || !PyType_Check(p[1]) || !PyDict_Check(p[2])) {
        PyErr_SetString(PyExc_TypeError, "setup(Desc, Job, addresses)");
        return nullptr;
    }
#define AQSGD_TAKE(name)                                                              \
    {                                                                                 \
        PyObject* a = PyDict_GetItemString(p[2], "aqsgd_" #name);                     \
        void* f = a ? PyLong_AsVoidPtr(a) : nullptr;                                  \
        if (!f) {                                                                     \
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, "aqsgd_" #name);   \
            return nullptr;                                                           \
        }                                                                             \
        g_api.name = reinterpret_cast<decltype(g_api.name)>(f);                       \
    }
    AQSGD_TAKE(codes_bytes) AQSGD_TAKE(scales_count) AQSGD_TAKE(lowbit_row_bytes) AQSGD_TAKE(topk_bitmap_bytes)
    AQSGD_TAKE(topk_codes_bytes) AQSGD_TAKE(encode) AQSGD_TAKE(decode) AQSGD_TAKE(grad_quant)
    AQSGD_TAKE(grad_dequant) AQSGD_TAKE(seed) AQSGD_TAKE(encode_seen) AQSGD_TAKE(decode_seen)
    AQSGD_TAKE(encode_lowbit) AQSGD_TAKE(decode_lowbit) AQSGD_TAKE(grad_topk_quant)
    AQSGD_TAKE(grad_topk_dequant) AQSGD_TAKE(run_jobs)
#undef AQSGD_TAKE
    Py_INCREF(p[0]);
    Py_INCREF(p[1]);
    g_desc_type = reinterpret_cast<PyTypeObject*>(p[0]);
    g_job_type = reinterpret_cast<PyTypeObject*>(p[1]);
    Py_RETURN_NONE;
}

#define AQSGD_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    AQSGD_METHOD(setup), AQSGD_METHOD(encode), AQSGD_METHOD(decode), AQSGD_METHOD(grad_quant),
    AQSGD_METHOD(grad_dequant), AQSGD_METHOD(seed), AQSGD_METHOD(encode_seen), AQSGD_METHOD(decode_seen),
    AQSGD_METHOD(encode_lowbit), AQSGD_METHOD(decode_lowbit), AQSGD_METHOD(grad_topk_quant),
    AQSGD_METHOD(grad_topk_dequant), AQSGD_METHOD(encode_job), AQSGD_METHOD(decode_job),
    AQSGD_METHOD(grad_quant_job), AQSGD_METHOD(grad_dequant_job), AQSGD_METHOD(run_jobs),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "The binding's per-call work (see binding.py).", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
