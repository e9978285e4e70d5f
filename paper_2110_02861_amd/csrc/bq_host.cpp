// Host side of the Python binding in native code: the module _bqhost.
//
// bq.py and optim.py describe each call completely and stay the reference for
// it: they check the arguments, name the errors, allocate the outputs and make
// the C call.  The functions here do the same for the ordinary case -- plain
// GPU tensors of the right type, size and device, all checks passing -- and
// return None for anything else, whereupon the Python code runs as if they
// did not exist.  Nothing is remembered between calls.
//
// Why: a call's Python took 8 to 10 us and a replayed optimizer step 0.5 us per
// param, more than the GPU needs for small arrays and for lists of many small
// tensors.  Measured, many calls in a row, without and with this module: quantize +
// dequantize of 300,007 values 21.8 and 8.1 us; replayed steps of the drop-in momentum
// on the ResNet-50 list (161 tensors) 90.4 and 57.5 us, which is the kernel's time, and
// of the drop-in Adam on 6 small tensors 21.2 and 13.6 us.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <initializer_list>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include "bq.h"

namespace {

// Entry points of the libbq.so that bq.py loaded (addresses passed to bind).
struct Library {
    decltype(&bq_quantize_blockwise) quantize;
    decltype(&bq_quantize_blockwise_prepared) quantize_prepared;
    decltype(&bq_dequantize_blockwise) dequantize;
    decltype(&bq_estimate_quantile_codebook) estimate;
    decltype(&bq_quantile_workspace_bytes) workspace_bytes;
    decltype(&bq_optimizer8bit_step) step;
    decltype(&bq_step_plan_run) run;
    decltype(&bq_step_plan_run_prepared) run_prepared;
} lib;

// Thrown where the Python code is to run instead (errors and unusual
// arguments included).
struct NotHandled {};

void need(bool ok)
{
    if (!ok)
        throw NotHandled{};
}

PyObject *none()
{
    Py_RETURN_NONE;
}

// Calls that are left to Python as a matter of course, found without a throw
// (which takes 2 us).
//
// The call may be intercepted by a Python mode (fake tensors, a default device,
// ...), which only the Python code goes through.
bool modes()
{
    return c10::impl::TorchDispatchModeTLS::any_modes_set() ||
           at::impl::PythonTorchFunctionTLS::stack_len() != 0;
}

// Whether every argument is None or of exactly torch's own classes.
bool plain(std::initializer_list<PyObject *> tensors)
{
    for (PyObject *o : tensors)
        if (o != Py_None && !THPVariable_CheckExact(o))
            return false;
    return true;
}

// A contiguous tensor of exactly torch's own classes on the current device.
const at::Tensor &tensor(PyObject *o, at::ScalarType type, int device)
{
    need(THPVariable_CheckExact(o));
    const at::Tensor &t = THPVariable_Unpack(o);
    need(t.is_cuda() && t.layout() == at::kStrided && t.scalar_type() == type &&
         t.get_device() == device && t.is_contiguous());
    return t;
}

const float *map_ptr(PyObject *o, int device)
{
    const at::Tensor &t = tensor(o, at::kFloat, device);
    need(t.numel() == 256);
    return static_cast<const float *>(t.data_ptr());
}

// A device buffer of any type.
void *buffer(PyObject *o, int64_t bytes, int device)
{
    need(THPVariable_CheckExact(o));
    const at::Tensor &t = THPVariable_Unpack(o);
    need(t.is_cuda() && t.layout() == at::kStrided && t.get_device() == device &&
         t.is_contiguous() && t.numel() * static_cast<int64_t>(t.element_size()) >= bytes);
    return t.data_ptr();
}

// An int, or any other object that stands for one (numpy's).
int64_t whole(PyObject *o)
{
    const long long v = PyLong_AsLongLong(o);  // by __index__
    if (v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        throw NotHandled{};
    }
    return v;
}

int32_t whole32(PyObject *o)
{
    const int64_t v = whole(o);
    need(v >= INT32_MIN && v <= INT32_MAX);
    return static_cast<int32_t>(v);
}

hipStream_t stream_of(PyObject *o, int device)
{
    if (o == Py_None)
        return c10::hip::getCurrentHIPStream(static_cast<c10::DeviceIndex>(device)).stream();
    PyObject *h = PyObject_GetAttrString(o, "cuda_stream");
    if (!h) {
        PyErr_Clear();
        throw NotHandled{};
    }
    void *p = PyLong_Check(h) ? PyLong_AsVoidPtr(h) : nullptr;
    const bool ok = PyLong_Check(h) && !PyErr_Occurred();
    Py_DECREF(h);
    PyErr_Clear();
    need(ok);
    return static_cast<hipStream_t>(p);
}

// A number of a hyperparameter dict, as ctypes converts it, or fallback where the
// key is absent and `required` is not set.
float number(PyObject *dict, const char *key, bool required, float fallback)
{
    PyObject *v = PyDict_GetItemString(dict, key);
    if (!v) {
        need(!required);
        return fallback;
    }
    const double d = PyFloat_AsDouble(v);
    if (d == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        throw NotHandled{};
    }
    return static_cast<float>(d);
}

bq_hparams hparams(PyObject *dict)
{
    need(PyDict_CheckExact(dict));
    bq_hparams h{};
    h.lr = number(dict, "lr", true, 0.0f);
    h.beta1 = number(dict, "beta1", true, 0.0f);
    h.beta2 = number(dict, "beta2", false, 0.0f);
    h.eps = number(dict, "eps", false, 0.0f);
    h.weight_decay = PyDict_GetItemString(dict, "wd") ? number(dict, "wd", true, 0.0f)
                                                      : number(dict, "weight_decay", false, 0.0f);
    PyObject *step = PyDict_GetItemString(dict, "step");
    need(step != nullptr);
    h.step = whole(step);
    h.trust_coeff = number(dict, "trust", false, 0.0f);
    return h;
}

// Runs f, which returns a new reference, and hands anything unusual to Python.
template <class F>
PyObject *handled(F f)
{
    try {
        return f();
    } catch (const NotHandled &) {
    } catch (const std::exception &) {
        // e.g. a tensor without storage: the Python code meets it again and
        // raises its error
    }
    PyErr_Clear();
    return none();
}

// The C call without the interpreter lock, as ctypes makes it (a launch waits
// when the queue is full).
template <class F>
bq_status unlocked(F f)
{
    PyThreadState *save = PyEval_SaveThread();
    const bq_status s = f();
    PyEval_RestoreThread(save);
    return s;
}

PyObject *status_or(bq_status s, PyObject *ok)
{
    if (s == BQ_OK)
        return ok;
    Py_DECREF(ok);
    return PyLong_FromLong(s);
}

// bind(addresses): the addresses of lib's entry points, in its order.
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 1 || !PyTuple_CheckExact(args[0]) || PyTuple_GET_SIZE(args[0]) != 8) {
        PyErr_SetString(PyExc_TypeError, "bind takes a tuple of 8 addresses");
        return nullptr;
    }
    void *p[8];
    for (int i = 0; i < 8; ++i) {
        p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(args[0], i));
        if (!p[i]) {
            if (!PyErr_Occurred())
                PyErr_SetString(PyExc_ValueError, "null address");
            return nullptr;
        }
    }
    lib.quantize = reinterpret_cast<decltype(lib.quantize)>(p[0]);
    lib.quantize_prepared = reinterpret_cast<decltype(lib.quantize_prepared)>(p[1]);
    lib.dequantize = reinterpret_cast<decltype(lib.dequantize)>(p[2]);
    lib.estimate = reinterpret_cast<decltype(lib.estimate)>(p[3]);
    lib.workspace_bytes = reinterpret_cast<decltype(lib.workspace_bytes)>(p[4]);
    lib.step = reinterpret_cast<decltype(lib.step)>(p[5]);
    lib.run = reinterpret_cast<decltype(lib.run)>(p[6]);
    lib.run_prepared = reinterpret_cast<decltype(lib.run_prepared)>(p[7]);
    return none();
}

// quantize(prepared, map or tables, x, blocksize, codes, absmax, stream) ->
// (codes, absmax), a status, or None.
PyObject *quantize(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    return handled([&]() -> PyObject * {
        need(nargs == 7);
        if (modes() || !plain({args[1], args[2], args[4], args[5]}))
            return none();
        const bool prepared = args[0] == Py_True;
        const int device = c10::hip::current_device();
        const void *map;
        if (prepared) {
            map = buffer(args[1], BQ_PREPARED_CODEBOOK_BYTES, device);
        } else {
            map = map_ptr(args[1], device);
        }
        const at::Tensor &x = tensor(args[2], at::kFloat, device);
        const int32_t blocksize = whole32(args[3]);
        const int64_t n = x.numel();
        if (n == 0 || blocksize <= 0)
            return none();
        const int64_t blocks = (n + blocksize - 1) / blocksize;
        const hipStream_t stream = stream_of(args[6], device);
        at::Tensor codes, absmax;
        if (args[4] == Py_None)
            codes = at::empty({n}, x.options().dtype(at::kByte));
        else
            codes = tensor(args[4], at::kByte, device);
        if (args[5] == Py_None)
            absmax = at::empty({blocks}, x.options());
        else
            absmax = tensor(args[5], at::kFloat, device);
        need(codes.numel() >= n && absmax.numel() >= blocks);
        const float *xp = static_cast<const float *>(x.data_ptr());
        uint8_t *cp = static_cast<uint8_t *>(codes.data_ptr());
        float *ap = static_cast<float *>(absmax.data_ptr());
        const bq_status s = unlocked([&] {
            return prepared ? lib.quantize_prepared(map, xp, n, blocksize, cp, ap, stream)
                            : lib.quantize(static_cast<const float *>(map), xp, n, blocksize, cp,
                                           ap, stream);
        });
        if (s != BQ_OK)
            return PyLong_FromLong(s);
        PyObject *out = PyTuple_New(2);
        if (!out)
            return nullptr;
        if (args[4] == Py_None)
            PyTuple_SET_ITEM(out, 0, THPVariable_Wrap(codes));
        else
            PyTuple_SET_ITEM(out, 0, Py_NewRef(args[4]));
        if (args[5] == Py_None)
            PyTuple_SET_ITEM(out, 1, THPVariable_Wrap(absmax));
        else
            PyTuple_SET_ITEM(out, 1, Py_NewRef(args[5]));
        return out;
    });
}

// dequantize(map, codes, absmax, blocksize, out, stream) -> out, a status, or
// None.
PyObject *dequantize(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    return handled([&]() -> PyObject * {
        need(nargs == 6);
        if (modes() || !plain({args[0], args[1], args[2], args[4]}))
            return none();
        const int device = c10::hip::current_device();
        const float *map = map_ptr(args[0], device);
        const at::Tensor &codes = tensor(args[1], at::kByte, device);
        const at::Tensor &absmax = tensor(args[2], at::kFloat, device);
        const int32_t blocksize = whole32(args[3]);
        const int64_t n = codes.numel();
        if (n == 0 || blocksize <= 0)
            return none();
        need(absmax.numel() >= (n + blocksize - 1) / blocksize);
        const hipStream_t stream = stream_of(args[5], device);
        at::Tensor out;
        if (args[4] == Py_None)
            out = at::empty({n}, absmax.options());
        else
            out = tensor(args[4], at::kFloat, device);
        need(out.numel() >= n);
        const uint8_t *cp = static_cast<const uint8_t *>(codes.data_ptr());
        const float *ap = static_cast<const float *>(absmax.data_ptr());
        float *op = static_cast<float *>(out.data_ptr());
        const bq_status s =
            unlocked([&] { return lib.dequantize(map, cp, ap, n, blocksize, op, stream); });
        if (s != BQ_OK)
            return PyLong_FromLong(s);
        return args[4] == Py_None ? THPVariable_Wrap(out) : Py_NewRef(args[4]);
    });
}

// estimate(x, out, workspace, stream), both buffers given -> out, a status, or
// None.
PyObject *estimate(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    return handled([&]() -> PyObject * {
        need(nargs == 4);
        if (modes() || !plain({args[0], args[1], args[2]}))
            return none();
        const int device = c10::hip::current_device();
        const at::Tensor &x = tensor(args[0], at::kFloat, device);
        const at::Tensor &out = tensor(args[1], at::kFloat, device);
        const int64_t n = x.numel();
        need(n > 0 && out.numel() == 256);
        void *wp = buffer(args[2], lib.workspace_bytes(n), device);
        const hipStream_t stream = stream_of(args[3], device);
        const float *xp = static_cast<const float *>(x.data_ptr());
        float *op = static_cast<float *>(out.data_ptr());
        const bq_status s = unlocked([&] { return lib.estimate(xp, n, wp, op, stream); });
        return status_or(s, Py_NewRef(args[1]));
    });
}

// run(handle, hp, map 1, map 2 or None, stream) -> a status or None.
PyObject *run(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    return handled([&]() -> PyObject * {
        need(nargs == 5);
        if (modes() || !plain({args[2], args[3]}))
            return none();
        const bq_step_plan plan = static_cast<bq_step_plan>(PyLong_AsVoidPtr(args[0]));
        need(plan != nullptr);
        const bq_hparams h = hparams(args[1]);
        const int device = c10::hip::current_device();
        const float *q1 = map_ptr(args[2], device);
        const float *q2 = args[3] == Py_None ? nullptr : map_ptr(args[3], device);
        const hipStream_t stream = stream_of(args[4], device);
        return PyLong_FromLong(unlocked([&] { return lib.run(plan, &h, q1, q2, stream); }));
    });
}

// run_prepared(handle, bytes needed, hp, prepared, stream) -> a status or None.
PyObject *run_prepared(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    return handled([&]() -> PyObject * {
        need(nargs == 5);
        if (modes() || !plain({args[3]}))
            return none();
        const bq_step_plan plan = static_cast<bq_step_plan>(PyLong_AsVoidPtr(args[0]));
        need(plan != nullptr);
        const bq_hparams h = hparams(args[2]);
        const int device = c10::hip::current_device();
        const at::Tensor &prepared = tensor(args[3], at::kByte, device);
        need(prepared.numel() >= whole(args[1]));
        const void *p = prepared.data_ptr();
        const hipStream_t stream = stream_of(args[4], device);
        return PyLong_FromLong(unlocked([&] { return lib.run_prepared(plan, &h, p, stream); }));
    });
}

// step(opt, blocksize, grad dtype, address of a bq_tensor array, count, hp,
// map 1, map 2 or None, stream) -> a status or None.
PyObject *step(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    return handled([&]() -> PyObject * {
        need(nargs == 9);
        if (modes() || !plain({args[6], args[7]}))
            return none();
        const int32_t opt = whole32(args[0]), blocksize = whole32(args[1]);
        const int32_t grad = whole32(args[2]), count = whole32(args[4]);
        const bq_tensor *list = static_cast<const bq_tensor *>(PyLong_AsVoidPtr(args[3]));
        need(list != nullptr);
        const bq_hparams h = hparams(args[5]);
        const int device = c10::hip::current_device();
        const float *q1 = map_ptr(args[6], device);
        const float *q2 = args[7] == Py_None ? nullptr : map_ptr(args[7], device);
        const hipStream_t stream = stream_of(args[8], device);
        return PyLong_FromLong(unlocked([&] {
            return lib.step(static_cast<bq_optimizer>(opt), blocksize,
                            static_cast<bq_dtype>(grad), list, count, &h, q1, q2, stream);
        }));
    });
}

// same_step(params, entries): whether a group's params with grads are those
// of a recorded step, in order, with every storage, type, size and state tensor
// as recorded (entries as optim.py makes them: param, its state, the state's
// first tensor, the param's and the grad's address, the grad's dtype, the
// number of elements).  None where a tensor is of another class than torch's or a
// torch mode is active.
PyObject *same_step(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    return handled([&]() -> PyObject * {
        need(nargs == 2 && PyList_CheckExact(args[0]) && PyList_CheckExact(args[1]));
        if (modes())
            return none();
        static PyObject *const kState1 = PyUnicode_InternFromString("state1");
        static PyObject *const kExpAvg = PyUnicode_InternFromString("exp_avg");
        PyObject *const params = args[0], *const entries = args[1];
        const Py_ssize_t n = PyList_GET_SIZE(entries);
        Py_ssize_t i = 0;
        for (Py_ssize_t k = 0; k < PyList_GET_SIZE(params); ++k) {
            PyObject *const o = PyList_GET_ITEM(params, k);
            if (!THPVariable_CheckExact(o))
                return none();
            const at::Tensor &p = THPVariable_Unpack(o);
            const at::Tensor &g = p.grad();
            if (!g.defined())
                continue;
            if (i == n)
                Py_RETURN_FALSE;
            PyObject *const e = PyList_GET_ITEM(entries, i);
            need(PyTuple_CheckExact(e) && PyTuple_GET_SIZE(e) == 7);
            PyObject *const state = PyTuple_GET_ITEM(e, 1);
            need(PyDict_CheckExact(state));
            // a grad of a subclass (it may have no Python object yet: then it
            // is a plain tensor)
            PyObject *const go = THPVariable_Wrap(g);
            need(go != nullptr);
            const bool exact = THPVariable_CheckExact(go);
            Py_DECREF(go);
            if (!exact)
                return none();
            if (PyTuple_GET_ITEM(e, 0) != o || g.layout() != at::kStrided ||
                reinterpret_cast<PyObject *>(torch::getTHPDtype(g.scalar_type())) !=
                    PyTuple_GET_ITEM(e, 5))
                Py_RETURN_FALSE;
            if (PyLong_AsVoidPtr(PyTuple_GET_ITEM(e, 3)) != p.data_ptr() ||
                PyLong_AsVoidPtr(PyTuple_GET_ITEM(e, 4)) != g.data_ptr())
                Py_RETURN_FALSE;
            const int64_t numel = whole(PyTuple_GET_ITEM(e, 6));
            if (g.numel() != numel || p.numel() != numel || !g.is_contiguous())
                Py_RETURN_FALSE;
            PyObject *s1 = PyDict_GetItem(state, kState1);
            if (!s1)
                s1 = PyDict_GetItem(state, kExpAvg);
            if (s1 != PyTuple_GET_ITEM(e, 2))
                Py_RETURN_FALSE;
            ++i;
        }
        if (i == n)
            Py_RETURN_TRUE;
        Py_RETURN_FALSE;
    });
}

// advance(entries): adds 1 to the step count of every entry's state.  True, or
// None (nothing changed) where a count is no plain int.
PyObject *advance(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    return handled([&]() -> PyObject * {
        need(nargs == 1 && PyList_CheckExact(args[0]));
        static PyObject *const kStep = PyUnicode_InternFromString("step");
        const Py_ssize_t n = PyList_GET_SIZE(args[0]);
        const auto state = [&](Py_ssize_t i) {
            PyObject *const e = PyList_GET_ITEM(args[0], i);
            need(PyTuple_CheckExact(e) && PyTuple_GET_SIZE(e) == 7 &&
                 PyDict_CheckExact(PyTuple_GET_ITEM(e, 1)));
            return PyTuple_GET_ITEM(e, 1);
        };
        for (Py_ssize_t i = 0; i < n; ++i) {
            PyObject *const v = PyDict_GetItem(state(i), kStep);
            need(v != nullptr && PyLong_CheckExact(v));
            need(whole(v) < INT64_MAX);
        }
        for (Py_ssize_t i = 0; i < n; ++i) {
            PyObject *const d = state(i);
            PyObject *const v = PyLong_FromLongLong(whole(PyDict_GetItem(d, kStep)) + 1);
            if (!v || PyDict_SetItem(d, kStep, v) != 0) {
                Py_XDECREF(v);
                return nullptr;  // out of memory
            }
            Py_DECREF(v);
        }
        Py_RETURN_TRUE;
    });
}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(bind), METH_FASTCALL, nullptr},
    {"quantize", reinterpret_cast<PyCFunction>(quantize), METH_FASTCALL, nullptr},
    {"dequantize", reinterpret_cast<PyCFunction>(dequantize), METH_FASTCALL, nullptr},
    {"estimate", reinterpret_cast<PyCFunction>(estimate), METH_FASTCALL, nullptr},
    {"run", reinterpret_cast<PyCFunction>(run), METH_FASTCALL, nullptr},
    {"run_prepared", reinterpret_cast<PyCFunction>(run_prepared), METH_FASTCALL, nullptr},
    {"step", reinterpret_cast<PyCFunction>(step), METH_FASTCALL, nullptr},
    {"same_step", reinterpret_cast<PyCFunction>(same_step), METH_FASTCALL, nullptr},
    {"advance", reinterpret_cast<PyCFunction>(advance), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bqhost", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bqhost() { return PyModule_Create(&module); }
