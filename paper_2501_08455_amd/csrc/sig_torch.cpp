// The torch side of the binding in native code: argument marshalling of the calls a program makes per batch
// (forward, gradient, row product) and the autograd node of the signature layer.  All arithmetic stays behind the C ABI
// (include/sig.h); this module only unpacks tensors, allocates results and finds the current stream.
//
// Small calls are bound by the host: four short paths take the GPU 3.7 us, and the same marshalling through ctypes and
// torch's Python layer took 9.7 us a call (forward and backward of a 128 x 100 x 5 mini-batch through
// torch.autograd.Function 106 us for 31 us of kernels).
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/python_variable.h>

#include "sig.h"

namespace {

using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

sig_ctx *default_ctx = nullptr;   // the binding's default context, set once by set_default_ctx

// A failed library call on its way to Python, where it becomes binding.SigError(status, where)
struct Failure {
    int status;
    const char *where;
};

// module.type(*args), raised; `args` is taken over
void raise_named(const char *module_name, const char *type_name, PyObject *args)
{
    PyObject *module = args ? PyImport_ImportModule(module_name) : nullptr;
    PyObject *type = module ? PyObject_GetAttrString(module, type_name) : nullptr;
    PyObject *error = type ? PyObject_CallObject(type, args) : nullptr;
    if (error) PyErr_SetObject(type, error);
    Py_XDECREF(error);
    Py_XDECREF(type);
    Py_XDECREF(module);
    Py_XDECREF(args);
}

PyObject *raise(const Failure &f)
{
    raise_named("paper_2501_08455_amd.binding", "SigError", Py_BuildValue("(is)", f.status, f.where));
    return nullptr;
}

// the same from a thread of the autograd engine: the exception travels as torch's carrier of Python errors
[[noreturn]] void rethrow_in_python(const Failure &f)
{
    const PyGILState_STATE gil = PyGILState_Ensure();
    python_error carrier;
    raise(f);
    carrier.persist();
    PyGILState_Release(gil);
    throw carrier;
}

void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// contiguous [B, L, d] of float32 on the GPU, as the library reads it
at::Tensor checked_path(const at::Tensor &path)
{
    if (!path.is_cuda() || path.scalar_type() != at::kFloat)
        throw std::invalid_argument("path must be a float32 tensor on the GPU");
    if (path.dim() != 3) throw std::invalid_argument("path must have three dimensions: batch, length, channels");
    return path.contiguous();
}

at::Tensor compute(const at::Tensor &x, int depth, bool stream)
{
    const int64_t B = x.size(0), L = x.size(1);
    const int d = (int)x.size(2);
    const int64_t D = sig_size(d, depth);
    if (D < 0) throw Failure{SIG_ERR_TOO_LARGE, "sig_size"};
    at::Tensor out = stream ? at::empty({B, L - 1, D}, x.options()) : at::empty({B, D}, x.options());
    const int rc = sig_compute(default_ctx, x.const_data_ptr<float>(), B, L, d, depth, stream, out.mutable_data_ptr<float>(),
                               current_stream());
    if (rc != SIG_OK) throw Failure{rc, "sig_compute"};
    return out;
}

// The layer as torch's C++ custom function: checkpointing, saved-tensor hooks and compiled autograd treat it as they treat a
// torch.autograd.Function, and the engine calls backward on its own thread without the interpreter lock.  (A bare
// torch::autograd::Node costs 2 us less of the 44 a small training step takes, and compiled autograd refuses it.)
struct Signature : torch::autograd::Function<Signature> {
    static at::Tensor forward(AutogradContext *ctx, const at::Tensor &path, int64_t depth, bool stream)
    {
        at::AutoDispatchBelowADInplaceOrView below_autograd;
        const at::Tensor x = checked_path(path);
        const at::Tensor out = compute(x, (int)depth, stream);
        ctx->save_for_backward({x, out});
        ctx->saved_data["depth"] = depth;
        ctx->saved_data["stream"] = stream;
        return out;
    }

    static variable_list backward(AutogradContext *ctx, const variable_list &grads)
    {
        const variable_list saved = ctx->get_saved_variables();
        const at::Tensor &x = saved[0], &y = saved[1];
        const int depth = (int)ctx->saved_data["depth"].toInt();
        at::AutoDispatchBelowADInplaceOrView below_autograd;
        const at::Tensor g = grads[0].contiguous();
        at::Tensor grad_path = at::empty_like(x);
        const int rc = sig_backward(default_ctx, x.const_data_ptr<float>(), x.size(0), x.size(1), (int)x.size(2), depth,
                                    ctx->saved_data["stream"].toBool(), y.const_data_ptr<float>(), g.const_data_ptr<float>(),
                                    grad_path.mutable_data_ptr<float>(), current_stream());
        if (rc != SIG_OK) rethrow_in_python(Failure{rc, "sig_backward"});
        return {grad_path, at::Tensor(), at::Tensor()};   // depth and stream have none
    }
};

at::Tensor differentiable_forward(const at::Tensor &path, int depth, bool stream)
{
    TORCH_CHECK_NOT_IMPLEMENTED(!path._fw_grad(0).defined(), "the signature has no forward-mode derivative");
    if (!torch::autograd::compute_requires_grad(path)) {   // nothing to record: the plain call (1.3 us of host time less)
        at::AutoDispatchBelowADInplaceOrView below_autograd;
        return compute(checked_path(path), depth, stream);
    }
    return Signature::apply(path, depth, stream);
}

// ---------------------------------------------------------------- Python arguments
const at::Tensor *tensor_arg(PyObject *o)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "expected a torch tensor, got %s", Py_TYPE(o)->tp_name);
        return nullptr;
    }
    return &THPVariable_Unpack(o);
}

// what int(o) gives
bool int_arg(PyObject *o, int *value)
{
    PyObject *number = PyLong_CheckExact(o) ? Py_NewRef(o) : PyNumber_Long(o);
    if (!number) return false;
    const long v = PyLong_AsLong(number);
    Py_DECREF(number);
    if (v == -1 && PyErr_Occurred()) return false;
    if (v != (long)(int)v) {
        PyErr_SetString(PyExc_OverflowError, "integer argument out of range");
        return false;
    }
    *value = (int)v;
    return true;
}

// a context or a stream: None, an address, or an object that holds one under `attribute`
bool address_arg(PyObject *o, const char *attribute, void **address)
{
    *address = nullptr;
    if (o == Py_None) return true;
    PyObject *value = PyLong_Check(o) ? Py_NewRef(o) : PyObject_GetAttrString(o, attribute);
    if (!value) return false;
    if (value != Py_None) *address = PyLong_AsVoidPtr(value);
    Py_DECREF(value);
    return !PyErr_Occurred();
}

bool stream_arg(PyObject *o, void **stream)
{
    if (o != Py_None) return address_arg(o, "cuda_stream", stream);
    *stream = current_stream();
    return true;
}

template <typename F>
PyObject *guarded(F f)
{
    try {
        return f();
    } catch (const Failure &e) {
        return raise(e);
    } catch (const std::invalid_argument &e) {
        PyErr_SetString(PyExc_ValueError, e.what());
    } catch (...) {
        // torch's own, and what Python code raised in between (python_error: a saved-tensor hook, a dispatch mode)
        torch::translate_exception_to_python(std::current_exception());
    }
    return nullptr;
}

// runs `f` without the interpreter lock (a launch may wait for room in the queue)
template <typename F>
auto unlocked(F f)
{
    struct Unlock {
        PyThreadState *state = PyEval_SaveThread();
        ~Unlock() { PyEval_RestoreThread(state); }
    } unlock;
    return f();
}

bool arity(Py_ssize_t n, Py_ssize_t want)
{
    if (n != want) PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return n == want;
}

template <bool DIFFERENTIABLE>
PyObject *py_signature(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    int depth;
    if (!arity(n, 3)) return nullptr;
    const at::Tensor *path = tensor_arg(args[0]);
    if (!path || !int_arg(args[1], &depth)) return nullptr;
    const int stream = PyObject_IsTrue(args[2]);
    if (stream < 0) return nullptr;
    return guarded([&] {
        at::Tensor out = unlocked([&] {
            if (DIFFERENTIABLE) return differentiable_forward(*path, depth, stream != 0);
            at::AutoDispatchBelowADInplaceOrView below_autograd;
            return compute(checked_path(*path), depth, stream != 0);
        });
        return THPVariable_Wrap(std::move(out));
    });
}

bool shape_of(const at::Tensor &path, int64_t *B, int64_t *L, int *d)
{
    if (path.dim() != 3) {
        PyErr_SetString(PyExc_ValueError, "path must have three dimensions: batch, length, channels");
        return false;
    }
    *B = path.size(0);
    *L = path.size(1);
    *d = (int)path.size(2);
    return true;
}

// (ctx, path, depth, stream_flag, out, stream) -> status
PyObject *py_compute(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    void *ctx, *st;
    int depth, flag, d;
    int64_t B, L;
    if (!arity(n, 6)) return nullptr;
    const at::Tensor *path = tensor_arg(args[1]), *out = path ? tensor_arg(args[4]) : nullptr;
    if (!out || !address_arg(args[0], "value", &ctx) || !int_arg(args[2], &depth) || !int_arg(args[3], &flag) ||
        !shape_of(*path, &B, &L, &d))
        return nullptr;
    return guarded([&]() -> PyObject * {
        if (!stream_arg(args[5], &st)) return nullptr;
        return PyLong_FromLong(unlocked([&] {
            return sig_compute((sig_ctx *)ctx, (const float *)path->const_data_ptr(), B, L, d, depth, flag,
                               (float *)out->mutable_data_ptr(), st);
        }));
    });
}

// (ctx, path, depth, stream_flag, out, grad_out, grad_path, stream) -> status
PyObject *py_backward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    void *ctx, *st;
    int depth, flag, d;
    int64_t B, L;
    if (!arity(n, 8)) return nullptr;
    const at::Tensor *t[4];
    const int at[4] = {1, 4, 5, 6};
    for (int i = 0; i < 4; ++i)
        if (!(t[i] = tensor_arg(args[at[i]]))) return nullptr;
    if (!address_arg(args[0], "value", &ctx) || !int_arg(args[2], &depth) || !int_arg(args[3], &flag) ||
        !shape_of(*t[0], &B, &L, &d))
        return nullptr;
    return guarded([&]() -> PyObject * {
        if (!stream_arg(args[7], &st)) return nullptr;
        return PyLong_FromLong(unlocked([&] {
            return sig_backward((sig_ctx *)ctx, (const float *)t[0]->const_data_ptr(), B, L, d, depth, flag,
                                (const float *)t[1]->const_data_ptr(), (const float *)t[2]->const_data_ptr(),
                                (float *)t[3]->mutable_data_ptr(), st);
        }));
    });
}

// (ctx, a, b, d, depth, out, stream) -> status
PyObject *py_combine(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    void *ctx, *st;
    int d, depth;
    if (!arity(n, 7)) return nullptr;
    const at::Tensor *a = tensor_arg(args[1]), *b = a ? tensor_arg(args[2]) : nullptr, *out = b ? tensor_arg(args[5]) : nullptr;
    if (!out || !address_arg(args[0], "value", &ctx) || !int_arg(args[3], &d) || !int_arg(args[4], &depth)) return nullptr;
    if (a->dim() < 1) {
        PyErr_SetString(PyExc_IndexError, "rows must have a batch dimension");
        return nullptr;
    }
    return guarded([&]() -> PyObject * {
        if (!stream_arg(args[6], &st)) return nullptr;
        return PyLong_FromLong(unlocked([&] {
            return sig_combine((sig_ctx *)ctx, (const float *)a->const_data_ptr(), (const float *)b->const_data_ptr(),
                               a->size(0), d, depth, (float *)out->mutable_data_ptr(), st);
        }));
    });
}

PyObject *py_set_default_ctx(PyObject *, PyObject *ctx)
{
    void *address;
    if (!address_arg(ctx, "value", &address)) return nullptr;
    default_ctx = (sig_ctx *)address;
    Py_RETURN_NONE;
}

#define FASTCALL(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL
PyMethodDef methods[] = {
    {"signature", FASTCALL(py_signature<false>), "signature(path, depth, stream): the default context, a new tensor"},
    {"autograd_signature", FASTCALL(py_signature<true>), "signature(path, depth, stream) with a gradient"},
    {"compute", FASTCALL(py_compute), "compute(ctx, path, depth, stream_flag, out, stream) -> status"},
    {"backward", FASTCALL(py_backward), "backward(ctx, path, depth, stream_flag, out, grad_out, grad_path, stream) -> status"},
    {"combine", FASTCALL(py_combine), "combine(ctx, a, b, d, depth, out, stream) -> status"},
    {"set_default_ctx", py_set_default_ctx, METH_O, "the context of signature and autograd_signature"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sig_torch", "native marshalling between torch and libsig", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__sig_torch() { return PyModule_Create(&module); }
