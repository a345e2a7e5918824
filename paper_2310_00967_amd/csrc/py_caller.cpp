// Marshalling of the Python binding's calls on a context: Caller.step,
// .ef_step and .sweep check the tensors, call the C ABI of
// include/micro_sparsify.h and wrap the results.  They take the plain case
// only (exact torch.Tensor buffers, Python floats and ints, every check
// passed) and return None otherwise, with nothing called: the Python methods
// then go their own way, which names what is wrong.  A nonzero status comes
// back as that int.  The C functions run without the interpreter lock, as
// ctypes runs them.
//
// In Python a step's checks, conversions and two views took 4.5 us of a call
// whose launch and wait take 12.
#include <Python.h>

#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>
#include <torch/torch.h>

#include <cstdint>

#include "micro_sparsify.h"

namespace {

struct Caller {
    PyObject_HEAD
    decltype(&micro_sparsify_step) step;
    decltype(&micro_ef_step) ef_step;
    decltype(&micro_sweep_step) sweep;
    micro_ctx* ctx;
    int64_t n_total;
    int device;
};

constexpr int kMaxSweepWorld = 64;

// The tensor of a plain 1-D contiguous buffer of the wanted type on the
// context's device with at least `least` values (exactly that many for
// `exact`), or null.
const at::Tensor* buffer(PyObject* o, const Caller* c, at::ScalarType type, int64_t least, bool exact) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (t.layout() != at::kStrided || t.scalar_type() != type || !t.is_cuda() || t.get_device() != c->device ||
        !t.is_contiguous())
        return nullptr;
    if (exact ? t.numel() != least : (t.dim() != 1 || t.numel() < least)) return nullptr;
    return &t;
}

bool integer(PyObject* o, int64_t* v) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &over);
    return over == 0;
}

bool real(PyObject* o, double* v) {
    if (!PyFloat_CheckExact(o)) return false;
    *v = PyFloat_AS_DOUBLE(o);
    return true;
}

struct Buffers {
    const at::Tensor *grad, *residual, *idx, *val;
};

bool buffers(const Caller* c, PyObject* grad, PyObject* residual, PyObject* idx, PyObject* val, int64_t capacity,
             Buffers* b) {
    b->grad = buffer(grad, c, at::kFloat, c->n_total, true);
    b->residual = buffer(residual, c, at::kFloat, c->n_total, true);
    b->idx = buffer(idx, c, at::kInt, capacity, false);
    b->val = buffer(val, c, at::kFloat, capacity, false);
    return b->grad && b->residual && b->idx && b->val;
}

int64_t partition_length(int64_t n, int64_t rank, int64_t world) {
    return (rank + 1) * n / world - rank * n / world;
}

// Views of the first k pairs, or false with the Python error set.
struct Pairs {
    THPObjectPtr idx, val;
    bool make(const Buffers& b, int64_t k) {
        idx = THPVariable_Wrap(b.idx->slice(0, 0, k));
        if (!idx.get()) return false;
        val = THPVariable_Wrap(b.val->slice(0, 0, k));
        return val.get() != nullptr;
    }
};

// A list of n new objects from make(i), or null with the Python error set.
template <class Make>
PyObject* list_of(int64_t n, Make make) {
    THPObjectPtr list(PyList_New(n));
    if (!list.get()) return nullptr;
    for (int64_t i = 0; i < n; ++i) {
        PyObject* item = make(i);
        if (!item) return nullptr;
        PyList_SET_ITEM(list.get(), i, item);
    }
    return list.release();
}

// step(grad, residual, rank, world, density, theta, out_idx, out_val)
PyObject* caller_step(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    Caller* c = reinterpret_cast<Caller*>(self);
    int64_t rank, world;
    double density, theta;
    Buffers b;
    HANDLE_TH_ERRORS
    if (n != 8 || !integer(args[2], &rank) || !integer(args[3], &world) || world < 1 || world > INT32_MAX ||
        rank < 0 || rank >= world || !real(args[4], &density) || !real(args[5], &theta) ||
        !buffers(c, args[0], args[1], args[6], args[7], partition_length(c->n_total, rank, world), &b))
        Py_RETURN_NONE;
    const float* grad = static_cast<const float*>(b.grad->data_ptr());
    float* residual = static_cast<float*>(b.residual->data_ptr());
    int32_t* idx = static_cast<int32_t*>(b.idx->data_ptr());
    float* val = static_cast<float*>(b.val->data_ptr());
    int64_t k = 0;
    micro_status st;
    Py_BEGIN_ALLOW_THREADS
    st = c->step(c->ctx, grad, residual, static_cast<int32_t>(rank), static_cast<int32_t>(world), density, &theta,
                 idx, val, &k);
    Py_END_ALLOW_THREADS
    if (st != MICRO_OK) return PyLong_FromLong(st);
    Pairs p;
    if (!p.make(b, k)) return nullptr;
    return Py_BuildValue("(LdOO)", static_cast<long long>(k), theta, p.idx.get(), p.val.get());
    END_HANDLE_TH_ERRORS
}

// ef_step(grad, residual, t, worker, world, density, theta, out_idx, out_val, local_error)
PyObject* caller_ef_step(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    Caller* c = reinterpret_cast<Caller*>(self);
    int64_t t, worker, world;
    double density, theta, sumsq = 0.0;
    Buffers b;
    HANDLE_TH_ERRORS
    if (n != 10 || !integer(args[2], &t) || !integer(args[3], &worker) || !integer(args[4], &world) || t < 0 ||
        world < 1 || world > INT32_MAX || worker < 0 || worker >= world || !real(args[5], &density) ||
        !real(args[6], &theta) || !PyBool_Check(args[9]))
        Py_RETURN_NONE;
    const int64_t part = (t % world + worker) % world;
    if (!buffers(c, args[0], args[1], args[7], args[8], partition_length(c->n_total, part, world), &b))
        Py_RETURN_NONE;
    const float* grad = static_cast<const float*>(b.grad->data_ptr());
    float* residual = static_cast<float*>(b.residual->data_ptr());
    int32_t* idx = static_cast<int32_t*>(b.idx->data_ptr());
    float* val = static_cast<float*>(b.val->data_ptr());
    const bool error = args[9] == Py_True;
    int64_t k = 0;
    int32_t cycle = 0;
    micro_status st;
    Py_BEGIN_ALLOW_THREADS
    st = c->ef_step(c->ctx, grad, residual, t, static_cast<int32_t>(worker), static_cast<int32_t>(world), density,
                    &theta, idx, val, &k, &cycle, error ? &sumsq : nullptr);
    Py_END_ALLOW_THREADS
    if (st != MICRO_OK) return PyLong_FromLong(st);
    Pairs p;
    if (!p.make(b, k)) return nullptr;
    if (error)
        return Py_BuildValue("(LdiOOd)", static_cast<long long>(k), theta, cycle, p.idx.get(), p.val.get(), sumsq);
    return Py_BuildValue("(LdiOO)", static_cast<long long>(k), theta, cycle, p.idx.get(), p.val.get());
    END_HANDLE_TH_ERRORS
}

// sweep(grad, residual, world, density, thetas, out_idx, out_val, want_sumsq)
PyObject* caller_sweep(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    Caller* c = reinterpret_cast<Caller*>(self);
    int64_t world, k[kMaxSweepWorld], total = 0;
    double density, theta[kMaxSweepWorld], sumsq[kMaxSweepWorld];
    Buffers b;
    HANDLE_TH_ERRORS
    if (n != 8 || !integer(args[2], &world) || world < 1 || world > kMaxSweepWorld || !real(args[3], &density) ||
        !PyList_CheckExact(args[4]) || PyList_GET_SIZE(args[4]) != world || !PyBool_Check(args[7]))
        Py_RETURN_NONE;
    for (int64_t r = 0; r < world; ++r)
        if (!real(PyList_GET_ITEM(args[4], r), &theta[r])) Py_RETURN_NONE;
    if (!buffers(c, args[0], args[1], args[5], args[6], c->n_total, &b)) Py_RETURN_NONE;
    const float* grad = static_cast<const float*>(b.grad->data_ptr());
    float* residual = static_cast<float*>(b.residual->data_ptr());
    int32_t* idx = static_cast<int32_t*>(b.idx->data_ptr());
    float* val = static_cast<float*>(b.val->data_ptr());
    const bool error = args[7] == Py_True;
    micro_status st;
    Py_BEGIN_ALLOW_THREADS
    st = c->sweep(c->ctx, grad, residual, static_cast<int32_t>(world), density, theta, idx, val, k,
                  error ? sumsq : nullptr);
    Py_END_ALLOW_THREADS
    if (st != MICRO_OK) return PyLong_FromLong(st);
    for (int64_t r = 0; r < world; ++r) total += k[r];
    THPObjectPtr ks(list_of(world, [&](int64_t r) { return PyLong_FromLongLong(k[r]); }));
    if (!ks.get()) return nullptr;
    THPObjectPtr ths(list_of(world, [&](int64_t r) { return PyFloat_FromDouble(theta[r]); }));
    if (!ths.get()) return nullptr;
    THPObjectPtr sqs(error ? list_of(world, [&](int64_t r) { return PyFloat_FromDouble(sumsq[r]); })
                           : Py_NewRef(Py_None));
    if (!sqs.get()) return nullptr;
    Pairs p;
    if (!p.make(b, total)) return nullptr;
    return Py_BuildValue("(OOOOO)", ks.get(), ths.get(), sqs.get(), p.idx.get(), p.val.get());
    END_HANDLE_TH_ERRORS
}

// Caller(step, ef_step, sweep, ctx, n_total, device): the C functions' and the
// context's addresses, the vector's length and the device's index.
PyObject* caller_new(PyTypeObject* type, PyObject* args, PyObject*) {
    unsigned long long step, ef_step, sweep, ctx;
    long long n_total;
    int device;
    if (!PyArg_ParseTuple(args, "KKKKLi", &step, &ef_step, &sweep, &ctx, &n_total, &device)) return nullptr;
    Caller* c = reinterpret_cast<Caller*>(type->tp_alloc(type, 0));
    if (!c) return nullptr;
    c->step = reinterpret_cast<decltype(c->step)>(step);
    c->ef_step = reinterpret_cast<decltype(c->ef_step)>(ef_step);
    c->sweep = reinterpret_cast<decltype(c->sweep)>(sweep);
    c->ctx = reinterpret_cast<micro_ctx*>(ctx);
    c->n_total = n_total;
    c->device = device;
    return reinterpret_cast<PyObject*>(c);
}

PyMethodDef caller_methods[] = {
    {"step", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(caller_step)), METH_FASTCALL, nullptr},
    {"ef_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(caller_ef_step)), METH_FASTCALL, nullptr},
    {"sweep", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(caller_sweep)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyTypeObject caller_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_caller", nullptr, -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__caller() {
    caller_type.tp_name = "paper_2310_00967_amd._caller.Caller";
    caller_type.tp_basicsize = sizeof(Caller);
    caller_type.tp_flags = Py_TPFLAGS_DEFAULT;
    caller_type.tp_methods = caller_methods;
    caller_type.tp_new = caller_new;
    if (PyType_Ready(&caller_type) < 0) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (!m) return nullptr;
    if (PyModule_AddObject(m, "Caller", Py_NewRef(reinterpret_cast<PyObject*>(&caller_type))) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
