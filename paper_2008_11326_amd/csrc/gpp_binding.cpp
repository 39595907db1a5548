// gpp_binding.cpp -- native side of the Python binding: checks the tensors
// of a call, allocates what the caller left out and calls the C ABI
// (include/gpp.h).  The package's functions call it first; it returns
//   a tuple   the call's results,
//   an int    the gpp_status of a library call that failed,
//   None      whenever an argument is anything but the plain case (exact
//             torch.Tensor or Parameter objects of the right type, device,
//             shape and layout, Python ints): the caller then goes through
//             its own checks, which name what is wrong or accept the rest.
// It keeps no tensor and caches nothing about one.
//
// Why native: a call of the forward has 6 input tensors with seven checks
// each, three allocations, a stream query and a device guard; from Python
// that was 20-22 us per call, as long as a small problem's kernels, and 6 us
// per state of a batched call (17.7 ms for 3000 tiny states whose kernels
// take 0.06 ms).
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <new>
#include <vector>

#include "gpp.h"

namespace {

// The library's entry points, taken from the copy the package has loaded.
struct Entries {
    decltype(&gpp_sigma_fwd_workspace) fwd_workspace = nullptr;
    decltype(&gpp_sigma_fwd) fwd = nullptr;
    decltype(&gpp_sigma_fwd_noalloc) fwd_noalloc = nullptr;
    decltype(&gpp_sigma_qp) qp = nullptr;
    decltype(&gpp_sigma_bwd_workspace) bwd_workspace = nullptr;
    decltype(&gpp_sigma_bwd) bwd = nullptr;
    decltype(&gpp_sigma_batched) batched = nullptr;
} lib;

PyObject *g_parameter = nullptr;  // torch.nn.Parameter
PyObject *g_keys[6] = {};         // the input names, interned

// The tensor of a plain strided device tensor object, else nullptr.
const at::Tensor *plain(PyObject *o)
{
    if (!THPVariable_CheckExact(o) && (PyObject *)Py_TYPE(o) != g_parameter) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.has_storage() || t.is_conj() ||
        t.is_neg() || t.unsafeGetTensorImpl()->is_python_dispatch())
        return nullptr;
    return &t;
}

// Whether t is a contiguous tensor of this type, shape and device.
bool fits(const at::Tensor *t, at::ScalarType type, at::IntArrayRef shape, at::Device dev)
{
    return t && t->scalar_type() == type && t->device() == dev && t->sizes() == shape &&
           t->is_contiguous();
}

template <typename T = double>
T *ptr(const at::Tensor &t)
{
    return t.numel() > 0 ? static_cast<T *>(t.data_ptr()) : nullptr;
}

bool small_int(PyObject *o, int64_t &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    v = PyLong_AsLongLongAndOverflow(o, &over);
    return !over;
}

struct Call {
    gpp_dims dims;
    gpp_inputs in;
    at::Device dev{at::kCPU};
};

constexpr auto kC = at::kComplexDouble;
constexpr auto kD = at::kDouble;

// The six inputs and nvband of one problem.
bool inputs(PyObject *const *o, int64_t nvband, Call &c)
{
    const at::Tensor *t[6];
    for (int i = 0; i < 6; ++i)
        if (!(t[i] = plain(o[i]))) return false;
    if (t[1]->dim() != 2 || t[2]->dim() != 2 || t[5]->dim() != 2) return false;
    const int64_t nb = t[1]->size(0), ng = t[1]->size(1), np = t[2]->size(0), nw = t[5]->size(0);
    c.dev = t[1]->device();
    if (!c.dev.is_cuda() || !fits(t[0], kC, {nb, ng}, c.dev) || !fits(t[1], kC, {nb, ng}, c.dev) ||
        !fits(t[2], kC, {np, ng}, c.dev) || !fits(t[3], kC, {np, ng}, c.dev) ||
        !fits(t[4], kD, {ng}, c.dev) || !fits(t[5], kD, {nw, nb}, c.dev))
        return false;
    c.dims = {nb, nvband, ng, np, nw};
    c.in = {ptr(*t[0]), ptr(*t[1]), ptr(*t[2]), ptr(*t[3]), ptr(*t[4]), ptr(*t[5])};
    return true;
}

// The stream argument: an int, or None for the current stream of dev.
bool stream_of(PyObject *o, at::Device dev, void *&s)
{
    if (o == Py_None) {
        s = c10::hip::getCurrentHIPStream(dev.index()).stream();
        return true;
    }
    int64_t v;
    if (!small_int(o, v)) return false;
    s = reinterpret_cast<void *>(v);
    return true;
}

at::Tensor make(at::IntArrayRef shape, at::ScalarType type, at::Device dev)
{
    return at::empty(shape, at::TensorOptions().dtype(type).device(dev));
}

// The caller's workspace, or one of `need` bytes.
bool workspace_of(PyObject *o, size_t need, at::Device dev, at::Tensor &w)
{
    if (o == Py_None) {
        w = make({(int64_t)need}, at::kByte, dev);
        return true;
    }
    const at::Tensor *t = plain(o);
    if (!t) return false;
    w = *t;
    return true;
}

// The caller's output tensors (a tuple or list of n), or new ones.
bool outputs_of(PyObject *o, int n, const at::ScalarType *type, const at::IntArrayRef *shape,
                at::Device dev, at::Tensor *out)
{
    if (o == Py_None) {
        for (int i = 0; i < n; ++i) out[i] = make(shape[i], type[i], dev);
        return true;
    }
    if (!PyTuple_CheckExact(o) && !PyList_CheckExact(o)) return false;
    if (PySequence_Fast_GET_SIZE(o) != n) return false;
    for (int i = 0; i < n; ++i) {
        const at::Tensor *t = plain(PySequence_Fast_GET_ITEM(o, i));
        if (!fits(t, type[i], shape[i], dev)) return false;
        out[i] = *t;
    }
    return true;
}

// The results as a tuple; undefined tensors (gradients not asked for) as
// None.  Objects the caller passed come back as themselves.
PyObject *results(gpp_status st, const at::Tensor *out, int n)
{
    if (st != GPP_OK) return PyLong_FromLong(st);
    PyObject *r = PyTuple_New(n);
    for (int i = 0; r && i < n; ++i) {
        PyObject *v = out[i].defined() ? THPVariable_Wrap(out[i]) : Py_NewRef(Py_None);
        if (!v) Py_CLEAR(r);
        else PyTuple_SET_ITEM(r, i, v);
    }
    return r;
}

// Runs fn; whatever it throws sends the call to the package's own checks.
template <typename F>
PyObject *guarded(F fn)
{
    try {
        PyObject *r = fn();
        if (!r) {
            if (PyErr_Occurred()) return nullptr;
            Py_RETURN_NONE;
        }
        return r;
    } catch (const std::exception &) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

template <typename F>
gpp_status without_gil(F fn)
{
    gpp_status st;
    Py_BEGIN_ALLOW_THREADS
    st = fn();
    Py_END_ALLOW_THREADS
    return st;
}

// fwd(6 inputs, nvband, out, workspace, stream)
PyObject *fwd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        int64_t nv;
        Call c;
        if (n != 10 || !lib.fwd || !small_int(a[6], nv) || !inputs(a, nv, c)) return nullptr;
        const int64_t nw = c.dims.nfreq;
        const at::ScalarType type[2] = {kC, kC};
        const at::IntArrayRef one(nw), shape[2] = {one, one};
        at::Tensor out[2], ws;
        void *stream;
        const size_t need = lib.fwd_workspace(&c.dims);
        if (!outputs_of(a[7], 2, type, shape, c.dev, out) ||
            !workspace_of(a[8], need ? need : 1, c.dev, ws) || !stream_of(a[9], c.dev, stream))
            return nullptr;
        const c10::DeviceGuard guard(c.dev);
        double *o0 = ptr(out[0]), *o1 = ptr(out[1]);
        void *w = ptr<void>(ws);
        const size_t wn = ws.numel();
        return results(without_gil([&] { return lib.fwd(&c.dims, &c.in, o0, o1, w, wn, stream); }),
                       out, 2);
    });
}

// fwd_noalloc(6 inputs, nvband, out, stream)
PyObject *fwd_noalloc(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        int64_t nv;
        Call c;
        if (n != 9 || !lib.fwd_noalloc || a[7] == Py_None || !small_int(a[6], nv) ||
            !inputs(a, nv, c))
            return nullptr;
        const int64_t nw = c.dims.nfreq;
        const at::ScalarType type[2] = {kC, kC};
        const at::IntArrayRef one(nw), shape[2] = {one, one};
        at::Tensor out[2];
        void *stream;
        if (!outputs_of(a[7], 2, type, shape, c.dev, out) || !stream_of(a[8], c.dev, stream))
            return nullptr;
        const c10::DeviceGuard guard(c.dev);
        double *o0 = ptr(out[0]), *o1 = ptr(out[1]);
        return results(without_gil([&] { return lib.fwd_noalloc(&c.dims, &c.in, o0, o1, stream); }),
                       out, 2);
    });
}

// qp(6 inputs, nvband, freq_step, energy, vxc, out, workspace, stream)
PyObject *qp(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        int64_t nv;
        Call c;
        if (n != 13 || !lib.qp || !small_int(a[6], nv) || !PyFloat_CheckExact(a[7]) ||
            !PyFloat_CheckExact(a[8]) || !PyFloat_CheckExact(a[9]) || !inputs(a, nv, c))
            return nullptr;
        const int64_t nw = c.dims.nfreq, six = 6;
        const at::ScalarType type[3] = {kC, kC, kD};
        const at::IntArrayRef one(nw), shape[3] = {one, one, at::IntArrayRef(six)};
        at::Tensor out[3], ws;
        void *stream;
        const size_t need = lib.fwd_workspace(&c.dims);
        if (!outputs_of(a[10], 3, type, shape, c.dev, out) ||
            !workspace_of(a[11], need ? need : 1, c.dev, ws) || !stream_of(a[12], c.dev, stream))
            return nullptr;
        const c10::DeviceGuard guard(c.dev);
        const double step = PyFloat_AS_DOUBLE(a[7]), energy = PyFloat_AS_DOUBLE(a[8]),
                     vxc = PyFloat_AS_DOUBLE(a[9]);
        double *o0 = ptr(out[0]), *o1 = ptr(out[1]), *o2 = ptr(out[2]);
        void *w = ptr<void>(ws);
        const size_t wn = ws.numel();
        return results(without_gil([&] {
                           return lib.qp(&c.dims, &c.in, step, energy, vxc, o0, o1, o2, w, wn, stream);
                       }),
                       out, 3);
    });
}

// bwd(6 inputs, nvband, grad_achtemp, grad_asxtemp, want, workspace, stream)
PyObject *bwd(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        int64_t nv;
        Call c;
        if (n != 12 || !lib.bwd || !small_int(a[6], nv) || !PyTuple_CheckExact(a[9]) ||
            PyTuple_GET_SIZE(a[9]) != 4 || !inputs(a, nv, c))
            return nullptr;
        const int64_t nb = c.dims.number_bands, ng = c.dims.ncouls, np = c.dims.ngpown,
                      nw = c.dims.nfreq;
        const at::Tensor *ga = plain(a[7]), *gs = plain(a[8]);
        if (!fits(ga, kC, {nw}, c.dev) || !fits(gs, kC, {nw}, c.dev)) return nullptr;
        bool want[4];
        for (int i = 0; i < 4; ++i) {
            PyObject *o = PyTuple_GET_ITEM(a[9], i);
            if (!PyBool_Check(o)) return nullptr;
            want[i] = o == Py_True;
        }
        at::Tensor out[4], ws;
        for (int i = 0; i < 4; ++i)
            if (want[i]) out[i] = make({i < 2 ? nb : np, ng}, kC, c.dev);
        void *stream;
        const size_t need = lib.bwd_workspace(&c.dims);
        if (!workspace_of(a[10], need > 256 ? need : 256, c.dev, ws) ||
            !stream_of(a[11], c.dev, stream))
            return nullptr;
        const c10::DeviceGuard guard(c.dev);
        double *o[4];
        for (int i = 0; i < 4; ++i) o[i] = want[i] ? ptr(out[i]) : nullptr;
        const double *pa = ptr(*ga), *ps = ptr(*gs);
        void *w = ptr<void>(ws);
        const size_t wn = ws.numel();
        return results(without_gil([&] {
                           return lib.bwd(&c.dims, &c.in, pa, ps, o[0], o[1], o[2], o[3], w, wn, stream);
                       }),
                       out, 4);
    });
}

// batched(plan address, address of its gpp_dims array, count, workspace
// bytes, states, out, workspace, stream)
PyObject *batched(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        int64_t plan, dims_at, count, need;
        if (n != 8 || !lib.batched || !small_int(a[0], plan) || !small_int(a[1], dims_at) ||
            !small_int(a[2], count) || !small_int(a[3], need) || !plan || count < 1)
            return nullptr;
        if (!PyList_CheckExact(a[4]) && !PyTuple_CheckExact(a[4])) return nullptr;
        if (PySequence_Fast_GET_SIZE(a[4]) != count) return nullptr;
        const gpp_dims *dims = reinterpret_cast<const gpp_dims *>(dims_at);
        std::vector<gpp_inputs> in(count);
        at::Device dev(at::kCPU);
        for (int64_t s = 0; s < count; ++s) {
            PyObject *st = PySequence_Fast_GET_ITEM(a[4], s), *o[6];
            if (PyDict_CheckExact(st)) {
                for (int i = 0; i < 6; ++i)
                    if (!(o[i] = PyDict_GetItemWithError(st, g_keys[i]))) return nullptr;
            } else if (PyTuple_CheckExact(st) && PyTuple_GET_SIZE(st) == 6) {
                for (int i = 0; i < 6; ++i) o[i] = PyTuple_GET_ITEM(st, i);
            } else {
                return nullptr;
            }
            Call c;
            if (!inputs(o, dims[s].nvband, c)) return nullptr;
            if (c.dims.number_bands != dims[s].number_bands || c.dims.ncouls != dims[s].ncouls ||
                c.dims.ngpown != dims[s].ngpown || c.dims.nfreq != dims[s].nfreq)
                return nullptr;
            if (s == 0) dev = c.dev;
            else if (dev != c.dev) return nullptr;
            in[s] = c.in;
        }
        const int64_t sizes[2] = {count, dims[0].nfreq};
        const at::ScalarType type[2] = {kC, kC};
        const at::IntArrayRef one(sizes, 2), shape[2] = {one, one};
        at::Tensor out[2], ws;
        void *stream;
        if (!outputs_of(a[5], 2, type, shape, dev, out) ||
            !workspace_of(a[6], need > 256 ? need : 256, dev, ws) || !stream_of(a[7], dev, stream))
            return nullptr;
        const c10::DeviceGuard guard(dev);
        double *o0 = ptr(out[0]), *o1 = ptr(out[1]);
        void *w = ptr<void>(ws);
        const size_t wn = ws.numel();
        return results(without_gil([&] {
                           return lib.batched(reinterpret_cast<gpp_plan *>(plan), in.data(), o0, o1,
                                              w, wn, stream);
                       }),
                       out, 2);
    });
}

// bind(addresses of the seven entry points in Entries' order,
// torch.nn.Parameter)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 8) {
        PyErr_SetString(PyExc_TypeError, "bind takes 8 arguments");
        return nullptr;
    }
    void *p[7];
    for (int i = 0; i < 7; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "NULL entry point");
            return nullptr;
        }
    }
    lib.fwd_workspace = reinterpret_cast<decltype(lib.fwd_workspace)>(p[0]);
    lib.fwd = reinterpret_cast<decltype(lib.fwd)>(p[1]);
    lib.fwd_noalloc = reinterpret_cast<decltype(lib.fwd_noalloc)>(p[2]);
    lib.qp = reinterpret_cast<decltype(lib.qp)>(p[3]);
    lib.bwd_workspace = reinterpret_cast<decltype(lib.bwd_workspace)>(p[4]);
    lib.bwd = reinterpret_cast<decltype(lib.bwd)>(p[5]);
    lib.batched = reinterpret_cast<decltype(lib.batched)>(p[6]);
    Py_INCREF(a[7]);
    Py_XDECREF(g_parameter);
    g_parameter = a[7];
    Py_RETURN_NONE;
}

#define GPP_M(name) \
    {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {GPP_M(bind), GPP_M(fwd), GPP_M(fwd_noalloc), GPP_M(qp),
                         GPP_M(bwd),  GPP_M(batched), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void)
{
    const char *names[6] = {"aqsmtemp",     "aqsntemp", "I_eps_array",
                            "wtilde_array", "vcoul",    "wx_array"};
    for (int i = 0; i < 6; ++i)
        if (!(g_keys[i] = PyUnicode_InternFromString(names[i]))) return nullptr;
    return PyModule_Create(&module);
}
