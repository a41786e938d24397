// The Python entry points' fast path (module _pqnative): checks and marshals tensors and enqueues through the C ABI.
//
// A scoring step over a small catalogue takes the GPU some 10 us; marshalled in Python (ctypes, torch.cuda.current_stream(),
// torch.empty(): about 2 us apiece) the same step took 28 us, most of it the interpreter.  Here a call costs well under a
// microsecond beside its kernel launches (about 3 us each in the HIP runtime).  No computation and no policy: whatever
// does not fit a function's plain case (a tensor that is not on the current device, of another type, not contiguous, a
// shape that disagrees) is answered with None, and binding.py's own code reports it.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/core/Allocator.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "pqtopk.h"

namespace {

PyObject* none() { Py_RETURN_NONE; }

// A contiguous tensor of that type on the current device, else nullptr.
const at::Tensor* plain(PyObject* o, at::ScalarType type, int device) {
    if (!THPVariable_Check(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.get_device() != device || t.scalar_type() != type || !t.is_contiguous()) return nullptr;
    return &t;
}

at::Tensor empty(at::IntArrayRef size, at::ScalarType type, int device) {
    return at::detail::empty_cuda(size, type, c10::Device(c10::DeviceType::CUDA, (c10::DeviceIndex)device), c10::nullopt);
}

void* current_stream() { return static_cast<void*>(c10::hip::getCurrentHIPStream().stream()); }

// The interpreter is free for other threads while the HIP runtime enqueues (it blocks when its queue is full).
template <typename F>
int without_gil(F&& f) {
    PyThreadState* t = PyEval_SaveThread();
    const int rc = f();
    PyEval_RestoreThread(t);
    return rc;
}

template <typename F>
PyObject* guarded(F&& f) {
    try {
        return f();
    } catch (const std::exception& e) {                       // (out of memory, mostly: torch's own words)
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// subitem_scores(queries, centroids, out | None) -> S, an error code (int), or None
PyObject* subitem_scores(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        if (n != 3) return none();
        const int device = c10::hip::current_device();
        const at::Tensor *q = plain(args[0], at::kFloat, device), *c = plain(args[1], at::kFloat, device);
        if (!q || !c || q->dim() != 2 || c->dim() != 3) return none();
        const int64_t B = q->size(0), d = q->size(1), m = c->size(0), b = c->size(1);
        if (m * c->size(2) != d) return none();
        PyObject* result = args[2];
        at::Tensor made;
        const at::Tensor* S;
        if (result == Py_None) {
            made = empty({B, m, b}, at::kFloat, device);
            S = &made;
            result = nullptr;
        } else {
            S = plain(result, at::kFloat, device);
            if (!S) return none();
        }
        const float *phi = q->const_data_ptr<float>(), *psi = c->const_data_ptr<float>();
        float* out = S->mutable_data_ptr<float>();
        void* st = current_stream();
        const int rc = without_gil([&]() { return pq_subitem_scores(phi, psi, out, (int)B, (int)d, (int)m, (int)b, st); });
        if (rc != PQ_OK) return PyLong_FromLong(rc);
        if (result) { Py_INCREF(result); return result; }
        return THPVariable_Wrap(std::move(made));
    });
}

// Outputs and workspace of a TopK call: the caller's, or made here.  The workspace made here is given back to torch's
// allocator when the call has been enqueued: memory freed on a stream is only handed out again behind the work enqueued there.
struct TopKBuffers {
    at::Tensor made_ids, made_scores;
    c10::DataPtr made_ws;
    const at::Tensor *ids = nullptr, *scores = nullptr;
    void* ws = nullptr;
    size_t ws_bytes = 0;

    template <typename Need>
    bool set(PyObject* ws_o, PyObject* ids_o, PyObject* scores_o, int64_t B, int64_t K, int device, Need&& need) {
        if (ids_o != Py_None && !(ids = plain(ids_o, at::kInt, device))) return false;
        if (scores_o != Py_None && !(scores = plain(scores_o, at::kFloat, device))) return false;
        if (ws_o != Py_None) {
            if (!THPVariable_Check(ws_o)) return false;
            const at::Tensor& t = THPVariable_Unpack(ws_o);
            ws = t.mutable_data_ptr();
            ws_bytes = (size_t)t.numel();
        } else {
            ws_bytes = need();
            if (ws_bytes < 16) ws_bytes = 16;
            made_ws = c10::GetAllocator(c10::DeviceType::CUDA)->allocate(ws_bytes);
            ws = made_ws.get();
        }
        if (!ids) { made_ids = empty({B, K}, at::kInt, device); ids = &made_ids; }
        if (!scores) { made_scores = empty({B, K}, at::kFloat, device); scores = &made_scores; }
        return true;
    }
    PyObject* result(PyObject* ids_o, PyObject* scores_o) {
        PyObject* i = ids_o != Py_None ? (Py_INCREF(ids_o), ids_o) : THPVariable_Wrap(std::move(made_ids));
        PyObject* s = scores_o != Py_None ? (Py_INCREF(scores_o), scores_o) : THPVariable_Wrap(std::move(made_scores));
        PyObject* r = PyTuple_New(2);
        PyTuple_SET_ITEM(r, 0, i);
        PyTuple_SET_ITEM(r, 1, s);
        return r;
    }
};

bool as_int(PyObject* o, int64_t* out) {
    if (!PyLong_Check(o)) return false;
    *out = PyLong_AsLongLong(o);
    if (*out == -1 && PyErr_Occurred()) { PyErr_Clear(); return false; }
    return *out >= 1 && *out <= PQ_MAX_K;                     // (anything else: the Python code's business)
}

// score_topk(codes, S, K, workspace | None, out_ids | None, out_scores | None) -> (ids, scores), an error code, or None
template <bool WIDE>
PyObject* score_topk(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        int64_t K;
        if (n != 6 || !as_int(args[2], &K)) return none();
        const int device = c10::hip::current_device();
        const at::Tensor *g = plain(args[0], WIDE ? at::kUInt16 : at::kByte, device), *S = plain(args[1], at::kFloat, device);
        if (!g || !S || g->dim() != 2 || S->dim() != 3) return none();
        const int64_t N = g->size(0), m = g->size(1), B = S->size(0), b = S->size(2);
        if (S->size(1) != m) return none();
        TopKBuffers io;
        auto need = [&]() { return WIDE ? pq_score_topk_u16_workspace_bytes(N, (int)B, (int)m, (int)b, (int)K)
                                        : pq_score_topk_workspace_bytes(N, (int)B, (int)m, (int)b, (int)K); };
        if (!io.set(args[3], args[4], args[5], B, K, device, need)) return none();
        int* ids = io.ids->mutable_data_ptr<int>();
        float *scores = io.scores->mutable_data_ptr<float>();
        const float* s = S->const_data_ptr<float>();
        const void* codes = g->const_data_ptr();
        void* st = current_stream();
        const int rc = without_gil([&]() {
            return WIDE ? pq_score_topk_u16(static_cast<const uint16_t*>(codes), s, N, (int)B, (int)m, (int)b, (int)K, ids, scores, io.ws,
                                            io.ws_bytes, st)
                        : pq_score_topk(static_cast<const uint8_t*>(codes), s, N, (int)B, (int)m, (int)b, (int)K, ids, scores, io.ws,
                                        io.ws_bytes, st);
        });
        if (rc != PQ_OK) return PyLong_FromLong(rc);
        return io.result(args[4], args[5]);
    });
}

// score_topk_subset(codes, S, subset, K, workspace | None, out_ids | None, out_scores | None) -> as score_topk
PyObject* score_topk_subset(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        int64_t K;
        if (n != 7 || !as_int(args[3], &K)) return none();
        const int device = c10::hip::current_device();
        const at::Tensor *g = plain(args[0], at::kByte, device), *S = plain(args[1], at::kFloat, device), *v = plain(args[2], at::kInt, device);
        if (!g || !S || !v || g->dim() != 2 || S->dim() != 3 || v->dim() != 1) return none();
        const int64_t N = g->size(0), m = g->size(1), B = S->size(0), b = S->size(2), nv = v->size(0);
        if (S->size(1) != m) return none();
        TopKBuffers io;
        if (!io.set(args[4], args[5], args[6], B, K, device,
                    [&]() { return pq_score_topk_subset_workspace_bytes(nv, (int)B, (int)m, (int)b, (int)K); }))
            return none();
        const uint8_t* codes = g->const_data_ptr<uint8_t>();
        const float* s = S->const_data_ptr<float>();
        const int* list = v->const_data_ptr<int>();
        int* ids = io.ids->mutable_data_ptr<int>();
        float* scores = io.scores->mutable_data_ptr<float>();
        void* st = current_stream();
        const int rc = without_gil([&]() {
            return pq_score_topk_subset(codes, s, list, nv, N, (int)B, (int)m, (int)b, (int)K, ids, scores, io.ws, io.ws_bytes, st);
        });
        if (rc != PQ_OK) return PyLong_FromLong(rc);
        return io.result(args[5], args[6]);
    });
}

// ---- Enqueue: an entry point with its arguments fixed; calling the object enqueues and returns `result`.  Base class of
// binding.py's Prepared classes, which keep the tensors alive and say what an error code means (`failed`).
enum Entry { kUnset, kSubitem, kTopK, kTopKU16, kTopKSubset };

struct Enqueue {
    PyObject_HEAD
    int entry;
    void *in0, *in1, *in2, *out0, *out1, *ws, *stream;
    long long N, n;
    size_t ws_bytes;
    int B, d, m, b, K;
    PyObject *result, *failed;
};

PyObject* enqueue_call(PyObject* self, PyObject*, PyObject*) {
    const Enqueue* e = reinterpret_cast<Enqueue*>(self);
    const int rc = without_gil([e]() -> int {
        const float* in1 = static_cast<const float*>(e->in1);
        int* ids = static_cast<int*>(e->out0);
        float* scores = static_cast<float*>(e->out1);
        switch (e->entry) {
            case kSubitem:
                return pq_subitem_scores(static_cast<const float*>(e->in0), in1, static_cast<float*>(e->out0), e->B, e->d, e->m, e->b, e->stream);
            case kTopK:
                return pq_score_topk(static_cast<const uint8_t*>(e->in0), in1, e->N, e->B, e->m, e->b, e->K, ids, scores, e->ws, e->ws_bytes,
                                     e->stream);
            case kTopKU16:
                return pq_score_topk_u16(static_cast<const uint16_t*>(e->in0), in1, e->N, e->B, e->m, e->b, e->K, ids, scores, e->ws,
                                         e->ws_bytes, e->stream);
            case kTopKSubset:
                return pq_score_topk_subset(static_cast<const uint8_t*>(e->in0), in1, static_cast<const int*>(e->in2), e->n, e->N, e->B, e->m,
                                            e->b, e->K, ids, scores, e->ws, e->ws_bytes, e->stream);
            default: return PQ_ERR_NULL;
        }
    });
    if (rc != PQ_OK) {
        if (e->failed) return PyObject_CallFunction(e->failed, "i", rc);
        PyErr_SetString(PyExc_RuntimeError, "called before it was prepared");
        return nullptr;
    }
    Py_INCREF(e->result);
    return e->result;
}

// _bind(entry, in0, in1, in2, n, N, B, d, m, b, K, out0, out1, ws, ws_bytes, stream, result, failed)
PyObject* enqueue_bind(PyObject* self, PyObject* args) {
    Enqueue* e = reinterpret_cast<Enqueue*>(self);
    int entry, B, d, m, b, K;
    unsigned long long in0, in1, in2, out0, out1, ws, ws_bytes, stream;
    long long n, N;
    PyObject *result, *failed;
    if (!PyArg_ParseTuple(args, "iKKKLLiiiiiKKKKKOO", &entry, &in0, &in1, &in2, &n, &N, &B, &d, &m, &b, &K, &out0, &out1, &ws, &ws_bytes,
                          &stream, &result, &failed))
        return nullptr;
    e->in0 = (void*)in0; e->in1 = (void*)in1; e->in2 = (void*)in2; e->out0 = (void*)out0; e->out1 = (void*)out1;
    e->ws = (void*)ws; e->ws_bytes = (size_t)ws_bytes; e->stream = (void*)stream;
    e->n = n; e->N = N; e->B = B; e->d = d; e->m = m; e->b = b; e->K = K;
    Py_INCREF(result);
    Py_INCREF(failed);
    Py_XSETREF(e->result, result);
    Py_XSETREF(e->failed, failed);
    e->entry = entry;
    Py_RETURN_NONE;
}

int enqueue_traverse(PyObject* self, visitproc visit, void* arg) {
    Enqueue* e = reinterpret_cast<Enqueue*>(self);
    Py_VISIT(e->result);
    Py_VISIT(e->failed);
    return 0;
}
int enqueue_clear(PyObject* self) {
    Enqueue* e = reinterpret_cast<Enqueue*>(self);
    e->entry = kUnset;
    Py_CLEAR(e->result);
    Py_CLEAR(e->failed);
    return 0;
}
void enqueue_dealloc(PyObject* self) {
    PyObject_GC_UnTrack(self);
    enqueue_clear(self);
    Py_TYPE(self)->tp_free(self);
}

PyMethodDef enqueue_methods[] = {{"_bind", enqueue_bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyTypeObject enqueue_type = {PyVarObject_HEAD_INIT(nullptr, 0) "_pqnative.Enqueue"};

PyMethodDef functions[] = {
    {"subitem_scores", (PyCFunction)(void (*)(void))subitem_scores, METH_FASTCALL, nullptr},
    {"score_topk", (PyCFunction)(void (*)(void))score_topk<false>, METH_FASTCALL, nullptr},
    {"score_topk_u16", (PyCFunction)(void (*)(void))score_topk<true>, METH_FASTCALL, nullptr},
    {"score_topk_subset", (PyCFunction)(void (*)(void))score_topk_subset, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pqnative", nullptr, -1, functions, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pqnative() {
    enqueue_type.tp_basicsize = sizeof(Enqueue);
    enqueue_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE | Py_TPFLAGS_HAVE_GC;
    enqueue_type.tp_new = PyType_GenericNew;
    enqueue_type.tp_call = enqueue_call;
    enqueue_type.tp_methods = enqueue_methods;
    enqueue_type.tp_traverse = enqueue_traverse;
    enqueue_type.tp_clear = enqueue_clear;
    enqueue_type.tp_dealloc = enqueue_dealloc;
    if (PyType_Ready(&enqueue_type) < 0) return nullptr;
    PyObject* mod = PyModule_Create(&module);
    if (!mod) return nullptr;
    Py_INCREF(&enqueue_type);
    PyModule_AddObject(mod, "Enqueue", reinterpret_cast<PyObject*>(&enqueue_type));
    PyModule_AddIntConstant(mod, "SUBITEM", kSubitem);
    PyModule_AddIntConstant(mod, "TOPK", kTopK);
    PyModule_AddIntConstant(mod, "TOPK_U16", kTopKU16);
    PyModule_AddIntConstant(mod, "TOPK_SUBSET", kTopKSubset);
    return mod;
}
