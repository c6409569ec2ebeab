// Argument marshalling of a hot call, for the Python binding: the same checks
// as bucket.py makes (type, dtype, element count, device, contiguity of every
// tensor), the pointer arrays on the stack and the library call, in one C
// call.  From Python each tensor costs about 0.7 us; a step over a bucket of
// 64 parameters took 180 us on the host for 16 us of kernels, and the toy
// block's four calls 51 us for 14.
//
// A call that does not pass every check here returns None and does nothing: the
// binding then goes through its own checks, which name what is wrong (or take
// what this module does not: tensor subclasses, lists that are not list or
// tuple, function modes).  Host code only; the library's functions come in as
// addresses, so whatever build of it the binding loaded is the one called.

#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "fsdp_bucket.h"

namespace {

// The library's hot functions, in the order of the addresses that the binding
// passes and of the `op` argument of a call.
enum Op { kAgPack, kAgUnpack, kRsPack, kRsReduce, kAgPackEx, kAgPackPush, kAgUnpackEx, kRsPackEx, kRsReduceEx, kOps };

struct Param {
    int64_t rows, inner, cpr, off, seg;      // N_p, inner_p, c_p, off_p, L_p
};

struct Caller {
    PyObject_HEAD
    std::vector<Param>* params;
    int64_t chunk;                   // S
    const fsdp_plan* plan;
    int32_t world;
    void* fn[kOps];
};

bool has_dtype(at::ScalarType t, fsdp_dtype code) {
    if (code == FSDP_DTYPE_BF16) return t == at::kBFloat16 || t == at::kShort || t == at::kUInt16;
    if (code == FSDP_DTYPE_F16) return t == at::kHalf;
    return t == at::kFloat || t == at::kInt;
}

// What one call's tensors have to share.
struct Checked {
    int device = -1;                 // of every non-empty tensor
    bool ok = true;
};

// The tensor's device pointer if it passes every check (NULL if it is empty).
// A bucket or a parameter may have any scalar type of its code, a shard
// (`fp32_only`) none but fp32.
void* pointer(PyObject* o, int64_t elems, fsdp_dtype code, bool fp32_only, Checked* c) {
    if (!THPVariable_CheckExact(o)) return c->ok = false, nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    const at::ScalarType type = t.scalar_type();
    if (fp32_only ? type != at::kFloat : !has_dtype(type, code)) return c->ok = false, nullptr;
    if (t.numel() != elems) return c->ok = false, nullptr;
    if (elems == 0) return nullptr;
    if (!t.is_cuda() || !t.is_contiguous() || !t.has_storage()) return c->ok = false, nullptr;
    const int device = t.device().index();
    if (c->device < 0) c->device = device;
    if (device != c->device) return c->ok = false, nullptr;
    return t.data_ptr();
}

struct Items {
    PyObject** at = nullptr;
    Py_ssize_t n = -1;
    explicit Items(PyObject* o) {
        if (PyList_CheckExact(o) || PyTuple_CheckExact(o)) {
            at = PySequence_Fast_ITEMS(o);
            n = PySequence_Fast_GET_SIZE(o);
        }
    }
};

// The bf16 / f32 / f16 code of a gradient list: every tensor's type must
// belong to the same one.
bool gradient_code(const Items& items, fsdp_dtype* code) {
    bool any = false;
    for (Py_ssize_t p = 0; p < items.n; ++p) {
        if (items.at[p] == Py_None) continue;
        if (!THPVariable_CheckExact(items.at[p])) return false;
        const at::ScalarType t = THPVariable_Unpack(items.at[p]).scalar_type();
        const fsdp_dtype c = has_dtype(t, FSDP_DTYPE_BF16) ? FSDP_DTYPE_BF16
                             : has_dtype(t, FSDP_DTYPE_F16) ? FSDP_DTYPE_F16 : FSDP_DTYPE_F32;
        if (any && c != *code) return false;
        *code = c;
        any = true;
    }
    if (!any) *code = FSDP_DTYPE_BF16;
    return true;
}

// run(op, rank, tensors, bucket, dtype, stream) -> status, or None when the
// call is left to the binding.  `tensors` are the per-parameter ones, `bucket`
// the bucket buffer (or the chunk list of the chunk forms), `dtype` the wire's
// code.
PyObject* run_checked(Caller* self, PyObject* const* args) {
    const long op = PyLong_AsLong(args[0]);
    const long rank = PyLong_CheckExact(args[1]) ? PyLong_AsLong(args[1]) : -1;
    const long wire = PyLong_AsLong(args[4]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    if (op < 0 || op >= kOps || wire < FSDP_DTYPE_BF16 || wire > FSDP_DTYPE_F16 || rank < 0 || rank >= self->world || self->plan == nullptr ||
        at::impl::torch_function_mode_enabled())
        Py_RETURN_NONE;
    const bool chunked = op >= kAgPackPush;
    const bool shards = op == kAgPack || op == kAgPackEx || op == kAgPackPush || op == kRsReduce || op == kRsReduceEx;
    const bool packed = op == kAgPack || op == kAgPackEx;           // one chunk
    const Items items(args[2]);
    const int P = int(self->params->size());
    if (items.n != P || P > FSDP_MAX_PARAMS) Py_RETURN_NONE;
    fsdp_dtype own = op == kRsPackEx ? FSDP_DTYPE_BF16 : fsdp_dtype(wire);
    if (op == kRsPackEx && !gradient_code(items, &own)) Py_RETURN_NONE;

    Checked c;
    void* tensors[FSDP_MAX_PARAMS];
    for (int p = 0; p < P; ++p) {
        const Param& q = (*self->params)[p];
        const int64_t held = shards ? std::min(q.cpr, std::max<int64_t>(0, q.rows - rank * q.cpr)) : q.rows;
        const int64_t elems = held * q.inner;
        if (items.at[p] == Py_None) {
            if (elems != 0) Py_RETURN_NONE;
            tensors[p] = nullptr;
            continue;
        }
        tensors[p] = pointer(items.at[p], elems, own, shards, &c);
        if (!c.ok) Py_RETURN_NONE;
    }
    void* buffer = nullptr;
    void* chunks[FSDP_MAX_CHUNKS];
    if (chunked) {
        const Items list(args[3]);
        if (list.n != self->world || self->world > FSDP_MAX_CHUNKS) Py_RETURN_NONE;
        for (int i = 0; i < self->world; ++i) {
            chunks[i] = pointer(list.at[i], self->chunk, fsdp_dtype(wire), false, &c);
            if (!c.ok) Py_RETURN_NONE;
        }
    } else {
        buffer = pointer(args[3], packed ? self->chunk : self->chunk * self->world, fsdp_dtype(wire), false, &c);
        if (!c.ok) Py_RETURN_NONE;
    }
    if (c.device < 0) Py_RETURN_NONE;                               // nothing but empty tensors

    hipStream_t stream;
    PyObject* const where = args[5];
    if (where == Py_None) {
        const auto current = c10::hip::getCurrentHIPStream();
        if (current.device_index() != c.device) Py_RETURN_NONE;
        stream = current.stream();
    } else {
        PyObject* handle = PyObject_GetAttrString(where, "cuda_stream");
        PyObject* device = handle ? PyObject_GetAttrString(where, "device") : nullptr;
        const bool fine = device && PyLong_Check(handle) && THPDevice_Check(device) &&
                          reinterpret_cast<THPDevice*>(device)->device.is_cuda() &&
                          reinterpret_cast<THPDevice*>(device)->device.index() == c.device;
        stream = fine ? static_cast<hipStream_t>(PyLong_AsVoidPtr(handle)) : nullptr;
        Py_XDECREF(handle);
        Py_XDECREF(device);
        PyErr_Clear();
        if (!fine) Py_RETURN_NONE;
    }

    const fsdp_plan* const plan = self->plan;
    void* const fn = self->fn[op];
    const int32_t r = int32_t(rank);
    const fsdp_dtype w = fsdp_dtype(wire);
    fsdp_status status = FSDP_OK;
    Py_BEGIN_ALLOW_THREADS
    switch (op) {
        case kAgPack:
            status = reinterpret_cast<decltype(&fsdp_ag_pack)>(fn)(plan, r, reinterpret_cast<const float* const*>(tensors),
                                                                    static_cast<uint16_t*>(buffer), stream);
            break;
        case kAgUnpack:
            status = reinterpret_cast<decltype(&fsdp_ag_unpack)>(fn)(plan, static_cast<const uint16_t*>(buffer),
                                                                      reinterpret_cast<uint16_t* const*>(tensors), stream);
            break;
        case kRsPack:
            status = reinterpret_cast<decltype(&fsdp_rs_pack)>(fn)(plan, reinterpret_cast<const uint16_t* const*>(tensors),
                                                                    static_cast<uint16_t*>(buffer), stream);
            break;
        case kRsReduce:
            status = reinterpret_cast<decltype(&fsdp_rs_reduce)>(fn)(plan, r, static_cast<const uint16_t*>(buffer),
                                                                      reinterpret_cast<float* const*>(tensors), stream);
            break;
        case kAgPackEx:
            status = reinterpret_cast<decltype(&fsdp_ag_pack_ex)>(fn)(plan, r, reinterpret_cast<const float* const*>(tensors),
                                                                       w, buffer, stream);
            break;
        case kAgPackPush:
            status = reinterpret_cast<decltype(&fsdp_ag_pack_push)>(fn)(plan, r, reinterpret_cast<const float* const*>(tensors),
                                                                         w, chunks, stream);
            break;
        case kAgUnpackEx:
            status = reinterpret_cast<decltype(&fsdp_ag_unpack_ex)>(fn)(plan, w, chunks, tensors, stream);
            break;
        case kRsPackEx:
            status = reinterpret_cast<decltype(&fsdp_rs_pack_ex)>(fn)(plan, own, tensors, w, chunks, stream);
            break;
        default:
            status = reinterpret_cast<decltype(&fsdp_rs_reduce_ex)>(fn)(plan, r, w, chunks,
                                                                         reinterpret_cast<float* const*>(tensors), stream);
    }
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

PyObject* caller_run(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    if (n != 6) {
        PyErr_SetString(PyExc_TypeError, "run takes 6 arguments");
        return nullptr;
    }
    try {
        return run_checked(reinterpret_cast<Caller*>(self), args);
    } catch (...) {
        // a tensor without plain storage, a stream query that failed, ...: the
        // binding's own path says what
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// Caller(plan, world, chunk, dims, addresses): `dims` is the list of (rows,
// inner) of the parameters, `addresses` the hot calls' and fsdp_plan_param's.
PyObject* caller_new(PyTypeObject* type, PyObject* args, PyObject*) {
    unsigned long long plan;
    int world;
    long long chunk;
    PyObject *dims, *fns;
    if (!PyArg_ParseTuple(args, "KiLO!O!", &plan, &world, &chunk, &PyList_Type, &dims, &PyTuple_Type, &fns))
        return nullptr;
    const Py_ssize_t P = PyList_GET_SIZE(dims);
    if (PyTuple_GET_SIZE(fns) != kOps + 1) {
        PyErr_SetString(PyExc_ValueError, "addresses of another library");
        return nullptr;
    }
    auto* self = reinterpret_cast<Caller*>(type->tp_alloc(type, 0));
    if (!self) return nullptr;
    self->plan = reinterpret_cast<const fsdp_plan*>(uintptr_t(plan));
    self->world = world;
    self->chunk = chunk;
    for (int k = 0; k < kOps; ++k) self->fn[k] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(fns, k));
    const auto query = reinterpret_cast<decltype(&fsdp_plan_param)>(PyLong_AsVoidPtr(PyTuple_GET_ITEM(fns, kOps)));
    if (PyErr_Occurred()) {
        Py_DECREF(self);
        return nullptr;
    }
    try {
        self->params = new std::vector<Param>;
        self->params->reserve(size_t(P));
        for (Py_ssize_t p = 0; p < P; ++p) {
            long long rows, inner;
            if (!PyArg_ParseTuple(PyList_GET_ITEM(dims, p), "LL", &rows, &inner)) {
                Py_DECREF(self);
                return nullptr;
            }
            Param q{rows, inner, 0, 0, 0};
            if (query(self->plan, int32_t(p), &q.cpr, &q.off, &q.seg) != FSDP_OK) {
                Py_DECREF(self);
                PyErr_SetString(PyExc_ValueError, "unknown plan");
                return nullptr;
            }
            self->params->push_back(q);
        }
    } catch (...) {
        Py_DECREF(self);
        return PyErr_NoMemory();
    }
    return reinterpret_cast<PyObject*>(self);
}

// params() -> [(c_p, off_p, L_p)]
PyObject* caller_params(PyObject* o, PyObject*) {
    const auto& params = *reinterpret_cast<Caller*>(o)->params;
    PyObject* list = PyList_New(Py_ssize_t(params.size()));
    if (!list) return nullptr;
    for (size_t p = 0; p < params.size(); ++p) {
        PyObject* t = Py_BuildValue("(LLL)", static_cast<long long>(params[p].cpr), static_cast<long long>(params[p].off),
                                    static_cast<long long>(params[p].seg));
        if (!t) {
            Py_DECREF(list);
            return nullptr;
        }
        PyList_SET_ITEM(list, Py_ssize_t(p), t);
    }
    return list;
}

void caller_dealloc(PyObject* o) {
    auto* self = reinterpret_cast<Caller*>(o);
    delete self->params;
    Py_TYPE(o)->tp_free(o);
}

// After close() the plan's handle is not used again.
PyObject* caller_close(PyObject* self, PyObject*) {
    reinterpret_cast<Caller*>(self)->plan = nullptr;
    Py_RETURN_NONE;
}

PyMethodDef caller_methods[] = {
    {"run", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(caller_run)), METH_FASTCALL,
     "run(op, rank, tensors, bucket, dtype, stream) -> status, or None when nothing was done"},
    {"params", caller_params, METH_NOARGS, "(rows per rank, offset, segment elements) of every parameter"},
    {"close", caller_close, METH_NOARGS, "forget the plan"},
    {nullptr, nullptr, 0, nullptr}};

PyTypeObject caller_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "Argument marshalling of the hot calls.", -1, nullptr,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
    caller_type.tp_name = "paper_2411_00284_amd._marshal.Caller";
    caller_type.tp_basicsize = sizeof(Caller);
    caller_type.tp_flags = Py_TPFLAGS_DEFAULT;
    caller_type.tp_methods = caller_methods;
    caller_type.tp_new = caller_new;
    caller_type.tp_dealloc = caller_dealloc;
    if (PyType_Ready(&caller_type) < 0) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&caller_type);
    if (PyModule_AddObject(m, "Caller", reinterpret_cast<PyObject*>(&caller_type)) < 0) {
        Py_DECREF(&caller_type);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
