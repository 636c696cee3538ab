// Native route of the tensor conveniences (lift.py): the checks, the output
// and the C call of an ordinary scal / asum / dot / gemv / BlackScholes / MD
// call without knobs, without the interpreter in between.
//
// Each function takes the call only if everything about it is ordinary --
// plain contiguous GPU tensors of a supported type, matching sizes, Python
// numbers -- and otherwise returns None, upon which the binding's own code
// does (or refuses) the call.  The two routes make the same C calls on the
// same stream with the same workspace.
//
// A call on 4097 elements spent 11.2 us in the interpreter for a 2 us kernel:
// argument checks 3, stream and workspace look-ups 4, the output 1.4 and the
// ctypes call 3.8 us.  This way it takes 4.3 us, of which the launch is 2.2.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <vector>

namespace {

using Status = int;
struct Entry {  // the C entry points, as addresses from the loaded library
    Status (*scal)(int64_t, float, const float *, float *, const void *, void *);
    Status (*asum)(int64_t, int, const void *, int, int, void *, void *, size_t, const void *, void *);
    Status (*dot)(int64_t, int, const void *, const void *, int, int, void *, void *, size_t, const void *, void *);
    Status (*gemv)(int64_t, int64_t, float, int, const void *, int64_t, const float *, float, float *, int, const void *,
                   void *);
    Status (*gemv_ws)(int64_t, int64_t, float, int, const void *, int64_t, const float *, float, float *, int, void *, size_t,
                      const void *, void *);
    Status (*blackscholes)(int64_t, const float *, float, float, float, float, float *, const void *, void *);
    Status (*md)(int64_t, const float *, int64_t, const int32_t *, float, float, float, float *, const void *, void *);
    Status (*capture_workspace)(void *, void **);
    size_t (*workspace_bytes)(void);
} entry;

PyObject *raw_stream = nullptr;      // device index -> stream handle of the current stream
PyObject *make_workspace = nullptr;  // device -> the (device, stream) workspace tensor
PyObject *check_status = nullptr;    // (status, name): raises

// The tensor behind a plain torch.Tensor on a GPU, contiguous; else null.
const at::Tensor *gpu_tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o))
        return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.has_storage() && t.is_cuda() && t.layout() == at::kStrided && t.is_contiguous() ? &t : nullptr;
}

bool is_f32(const at::Tensor &t) { return t.scalar_type() == at::kFloat; }

// lift_dtype of a storage type, or -1.
int storage_code(const at::Tensor &t)
{
    switch (t.scalar_type()) {
    case at::kFloat: return 0;
    case at::kBFloat16: return 1;
    case at::kHalf: return 2;
    default: return -1;
    }
}

// lift_acc of the binding's names, or -1.
int acc_code(PyObject *o)
{
    if (!PyUnicode_CheckExact(o))
        return -1;
    if (PyUnicode_CompareWithASCIIString(o, "f32") == 0)
        return 0;
    if (PyUnicode_CompareWithASCIIString(o, "comp") == 0)
        return 1;
    if (PyUnicode_CompareWithASCIIString(o, "f64combine") == 0)
        return 2;
    return -1;
}

bool number(PyObject *o, float *out)
{
    if (PyFloat_CheckExact(o))
        *out = (float)PyFloat_AS_DOUBLE(o);
    else if (PyLong_CheckExact(o)) {
        const double v = PyLong_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) {
            PyErr_Clear();
            return false;
        }
        *out = (float)v;
    } else
        return false;
    return true;
}

// Handle of the current stream of t's device; false with an exception set.
bool current_stream(const at::Tensor &t, void **out)
{
    PyObject *dev = PyLong_FromLong(t.get_device());
    if (!dev)
        return false;
    PyObject *h = PyObject_CallOneArg(raw_stream, dev);
    Py_DECREF(dev);
    if (!h)
        return false;
    *out = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    return !PyErr_Occurred();
}

// The workspace of a call on a stream: the graph's own where the stream is
// being captured, else that of (device, stream), the binding's own, held here
// too so that the look-up of a stream met before is a short search.
struct Workspace {
    at::Tensor tensor;
    void *at = nullptr;
    size_t bytes = 0;
};

bool workspace(PyObject *tensor, const at::Tensor &t, void *stream, Workspace *out)
{
    struct Known {
        int64_t device;
        void *stream;
        at::Tensor tensor;
    };
    static std::vector<Known> *known = new std::vector<Known>();   // under the interpreter's lock
    const Status st = entry.capture_workspace(stream, &out->at);
    if (st != 0) {
        PyObject *r = PyObject_CallFunction(check_status, "is", st, "lift_capture_workspace");
        Py_XDECREF(r);
        if (r)
            PyErr_SetString(PyExc_RuntimeError, "lift_capture_workspace");
        return false;
    }
    if (out->at) {
        out->bytes = entry.workspace_bytes();
        return true;
    }
    const auto take = [&](const at::Tensor &ws) {
        out->tensor = ws;
        out->at = ws.data_ptr();
        out->bytes = (size_t)ws.numel();
        return true;
    };
    for (const Known &w : *known)
        if (w.stream == stream && w.device == t.get_device())
            return take(w.tensor);
    PyObject *dev = PyObject_GetAttrString(tensor, "device");
    if (!dev)
        return false;
    PyObject *ws = PyObject_CallOneArg(make_workspace, dev);
    Py_DECREF(dev);
    if (!ws)
        return false;
    if (known->size() == 64)       // more streams than that: the oldest is looked up again when it returns
        known->erase(known->begin());
    known->push_back({t.get_device(), stream, THPVariable_Unpack(ws)});
    Py_DECREF(ws);
    return take(known->back().tensor);
}

PyObject *none()
{
    Py_RETURN_NONE;
}

// `value` if the call succeeded, else the binding's exception for its status.
PyObject *finish(Status st, const char *name, PyObject *value)
{
    if (st == 0)
        return value;
    Py_XDECREF(value);
    PyObject *r = PyObject_CallFunction(check_status, "is", st, name);
    Py_XDECREF(r);
    if (r)
        PyErr_SetString(PyExc_RuntimeError, name);
    return nullptr;
}

// call() without the interpreter's lock, as ctypes makes it.
template <class F>
Status unlocked(F &&call)
{
    struct Lock {   // given back on the way out of an exception too
        PyThreadState *save = PyEval_SaveThread();
        ~Lock() { PyEval_RestoreThread(save); }
    } lock;
    return call();
}

PyObject *reduce(PyObject *xo, PyObject *yo, PyObject *acco, PyObject *dtype)
{
    const at::Tensor *x = gpu_tensor(xo), *y = yo ? gpu_tensor(yo) : nullptr;
    const int acc = acc_code(acco);
    if (!x || (yo && !y) || acc < 0)
        return none();
    const int code = storage_code(*x);
    if (code < 0 || (y && (y->scalar_type() != x->scalar_type() || y->numel() != x->numel() || y->device() != x->device())))
        return none();
    at::ScalarType rt = at::kFloat;
    if (dtype != Py_None) {
        if (!THPDtype_Check(dtype))
            return none();
        rt = reinterpret_cast<THPDtype *>(dtype)->scalar_type;
        if (rt != at::kFloat && rt != at::kDouble)
            return none();
    }
    void *stream = nullptr;
    Workspace ws;
    if (!current_stream(*x, &stream) || !workspace(xo, *x, stream, &ws))
        return nullptr;
    at::Tensor result;
    const Status st = unlocked([&] {
        const int64_t n = x->numel();
        const int rc = rt == at::kDouble ? 3 : 0;
        result = at::empty({}, x->options().dtype(rt).requires_grad(false));
        return y ? entry.dot(n, code, x->const_data_ptr(), y->const_data_ptr(), acc, rc, result.data_ptr(), ws.at, ws.bytes,
                             nullptr, stream)
                 : entry.asum(n, code, x->const_data_ptr(), acc, rc, result.data_ptr(), ws.at, ws.bytes, nullptr, stream);
    });
    return finish(st, y ? "lift_dot" : "lift_asum", st == 0 ? THPVariable_Wrap(std::move(result)) : nullptr);
}

// The call's output: the caller's tensor, or a new binary32 one of `shape` on
// like's device.  Null: the caller's is out of the ordinary.
struct Output {
    at::Tensor made;
    PyObject *given = nullptr;
    const at::Tensor *tensor = nullptr;

    Output(PyObject *out, const at::Tensor &like, at::IntArrayRef shape)
    {
        if (out == Py_None) {
            made = at::empty(shape, like.options().dtype(at::kFloat).requires_grad(false));
            tensor = &made;
        } else {
            given = out;
            tensor = gpu_tensor(out);
        }
    }
    bool fits(int64_t numel) const { return tensor && is_f32(*tensor) && tensor->numel() == numel; }
    float *data() const { return static_cast<float *>(tensor->data_ptr()); }
    PyObject *object()
    {
        if (!given)
            return THPVariable_Wrap(std::move(made));
        Py_INCREF(given);
        return given;
    }
};

PyObject *call_scal(PyObject *const *args)   // alpha, x, out
{
    float alpha;
    const at::Tensor *x = gpu_tensor(args[1]);
    if (!x || !number(args[0], &alpha) || !is_f32(*x))
        return none();
    Output out(args[2], *x, x->sizes());
    if (!out.fits(x->numel()))
        return none();
    void *stream;
    if (!current_stream(*x, &stream))
        return nullptr;
    const Status st = unlocked([&] {
        return entry.scal(x->numel(), alpha, x->const_data_ptr<float>(), out.data(), nullptr, stream);
    });
    return finish(st, "lift_scal", out.object());
}

PyObject *call_gemv(PyObject *const *args)   // alpha, A, x, beta, y, acc
{
    float alpha, beta;
    const at::Tensor *A = gpu_tensor(args[1]), *x = gpu_tensor(args[2]), *y = gpu_tensor(args[4]);
    const int acc = acc_code(args[5]);
    if (!A || !x || !y || acc < 0 || !number(args[0], &alpha) || !number(args[3], &beta))
        return none();
    const int code = storage_code(*A);
    if (code < 0 || A->dim() != 2 || !is_f32(*x) || !is_f32(*y))
        return none();
    const int64_t m = A->size(0), lda = A->size(1), cols = x->numel();
    if (lda < cols || y->numel() != m)
        return none();
    void *stream;
    if (!current_stream(*A, &stream))
        return nullptr;
    // few long rows are split through a workspace (the binding's own code takes
    // 12 us whatever the size; through here, bf16: 8 x 33000 6.4, 22 x 60184
    // 7.8, 8 x 65539 5.3 us)
    Workspace ws;
    if (cols * A->element_size() > 65536 && m <= 512 && !workspace(args[1], *A, stream, &ws))
        return nullptr;
    const Status st = unlocked([&] {
        if (ws.at)
            return entry.gemv_ws(m, cols, alpha, code, A->const_data_ptr(), lda, x->const_data_ptr<float>(), beta,
                                 static_cast<float *>(y->data_ptr()), acc, ws.at, ws.bytes, nullptr, stream);
        return entry.gemv(m, cols, alpha, code, A->const_data_ptr(), lda, x->const_data_ptr<float>(), beta,
                          static_cast<float *>(y->data_ptr()), acc, nullptr, stream);
    });
    Py_INCREF(args[4]);
    return finish(st, "lift_gemv", args[4]);
}

PyObject *call_blackscholes(PyObject *const *args)   // s, strike, rate, volatility, years, out
{
    float p[4];
    const at::Tensor *s = gpu_tensor(args[0]);
    if (!s || !is_f32(*s))
        return none();
    for (int i = 0; i < 4; ++i)
        if (!number(args[1 + i], &p[i]))
            return none();
    Output out(args[5], *s, {s->numel(), 2});
    if (!out.fits(2 * s->numel()))
        return none();
    void *stream;
    if (!current_stream(*s, &stream))
        return nullptr;
    const Status st = unlocked([&] {
        return entry.blackscholes(s->numel(), s->const_data_ptr<float>(), p[0], p[1], p[2], p[3],
                                  out.data(), nullptr, stream);
    });
    return finish(st, "lift_blackscholes", out.object());
}

PyObject *call_md(PyObject *const *args)   // pos, nbr, cutoff, epsilon, sigma, out
{
    float p[3];
    const at::Tensor *pos = gpu_tensor(args[0]), *nbr = gpu_tensor(args[1]);
    if (!pos || !nbr || !is_f32(*pos) || nbr->scalar_type() != at::kInt || pos->dim() != 2 || pos->size(1) != 4 ||
        nbr->dim() != 2 || nbr->size(0) != pos->size(0))
        return none();
    for (int i = 0; i < 3; ++i)
        if (!number(args[2 + i], &p[i]))
            return none();
    Output out(args[5], *pos, {pos->size(0), 4});
    if (!out.fits(4 * pos->size(0)))
        return none();
    void *stream;
    if (!current_stream(*pos, &stream))
        return nullptr;
    const Status st = unlocked([&] {
        return entry.md(pos->size(0), pos->const_data_ptr<float>(), nbr->size(1), nbr->const_data_ptr<int32_t>(), p[0], p[1],
                        p[2], out.data(), nullptr, stream);
    });
    return finish(st, "lift_md", out.object());
}

PyObject *call_asum(PyObject *const *args)   // x, acc, result dtype or None
{
    return reduce(args[0], nullptr, args[1], args[2]);
}

PyObject *call_dot(PyObject *const *args)   // x, y, acc, result dtype or None
{
    return reduce(args[0], args[1], args[2], args[3]);
}

// No C++ exception leaves an entry point: what the tensor library refuses
// here, the binding's own code meets (and reports) itself.
template <PyObject *(*F)(PyObject *const *), Py_ssize_t COUNT>
PyObject *guarded(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != COUNT)
        return none();
    try {
        return F(args);
    } catch (...) {
        return none();
    }
}

// init(addresses of scal_ex, asum_ex, dot_ex, gemv_ex, blackscholes_ex, md_ex, gemv_ex_ws, capture_workspace, workspace_bytes,
// raw_stream, workspace, check)
PyObject *init(PyObject *, PyObject *args)
{
    unsigned long long a[9];
    PyObject *s, *w, *c;
    if (!PyArg_ParseTuple(args, "KKKKKKKKKOOO", &a[0], &a[1], &a[2], &a[3], &a[4], &a[5], &a[6], &a[7], &a[8], &s, &w, &c))
        return nullptr;
    entry.scal = reinterpret_cast<decltype(entry.scal)>(a[0]);
    entry.asum = reinterpret_cast<decltype(entry.asum)>(a[1]);
    entry.dot = reinterpret_cast<decltype(entry.dot)>(a[2]);
    entry.gemv = reinterpret_cast<decltype(entry.gemv)>(a[3]);
    entry.blackscholes = reinterpret_cast<decltype(entry.blackscholes)>(a[4]);
    entry.md = reinterpret_cast<decltype(entry.md)>(a[5]);
    entry.gemv_ws = reinterpret_cast<decltype(entry.gemv_ws)>(a[6]);
    entry.capture_workspace = reinterpret_cast<decltype(entry.capture_workspace)>(a[7]);
    entry.workspace_bytes = reinterpret_cast<decltype(entry.workspace_bytes)>(a[8]);
    Py_INCREF(s);
    Py_INCREF(w);
    Py_INCREF(c);
    Py_XDECREF(raw_stream);
    Py_XDECREF(make_workspace);
    Py_XDECREF(check_status);
    raw_stream = s;
    make_workspace = w;
    check_status = c;
    return none();
}

template <PyObject *(*F)(PyObject *const *), Py_ssize_t COUNT>
PyCFunction method()
{
    return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<F, COUNT>));
}

PyMethodDef methods[] = {
    {"init", init, METH_VARARGS, nullptr},
    {"scal", method<call_scal, 3>(), METH_FASTCALL, nullptr},
    {"asum", method<call_asum, 3>(), METH_FASTCALL, nullptr},
    {"dot", method<call_dot, 4>(), METH_FASTCALL, nullptr},
    {"gemv", method<call_gemv, 6>(), METH_FASTCALL, nullptr},
    {"blackscholes", method<call_blackscholes, 6>(), METH_FASTCALL, nullptr},
    {"md", method<call_md, 6>(), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tensor_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// INTERFACE: of init(); the binding takes no other.
PyMODINIT_FUNC PyInit__tensor_calls()
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddIntConstant(m, "INTERFACE", 2) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
