// CPython module `_native`: the fast way from a Python call to the C ABI (include/lbp_wht.h).
//
// A small layer's kernels take a few microseconds, so what bounds such a call is the host.  Checking shapes,
// allocating outputs and marshalling pointers through ctypes took 11-12 us per call (out of 19-23 us for one
// ViT-B image); here the same steps take about 2.  Every function takes the arguments of its namesake in
// binding.py, positionally, and returns
//   the outputs        the call was made,
//   an int             the library's status code (binding.py raises for it),
//   None               an argument this module does not take (not a tensor, a wrong shape, dtype or device):
//                      binding.py goes through its own checks, which name the error.
// Nothing is computed here and nothing is kept between calls.  Arguments are read with the interpreter's lock held;
// memory is allocated and the library called without it: both can wait for the device (an allocation that has to
// free others first, a workspace that grows, a full launch queue), and what the device waits for may be a
// collective that a thread of another GPU has still to launch.
#include <Python.h>

#include <ATen/Functions.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/autocast_mode.h>
#include <ATen/core/Tensor.h>
#include <ATen/core/grad_mode.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/python_cpp_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/autograd/saved_variable.h>

#include "../../include/lbp_wht.h"

namespace {

constexpr int kMaxIdx = 256;

struct Bases {
    int32_t v[kMaxIdx];
    int n = 0;
};

bool read_int(PyObject *o, long *out)
{
    if (!PyLong_Check(o)) return false;
    int overflow = 0;
    *out = PyLong_AsLongAndOverflow(o, &overflow);
    return overflow == 0 && *out >= INT32_MIN && *out <= INT32_MAX;
}

// Any object is true or false; one that cannot say leaves its error set: false is returned.
bool read_truth(PyObject *o, bool *out)
{
    const int v = PyObject_IsTrue(o);
    *out = v > 0;
    return v >= 0;
}

bool read_bases(PyObject *o, Bases *b)
{
    if (!PyList_Check(o) && !PyTuple_Check(o)) return false;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
    if (n > kMaxIdx) return false;
    PyObject **items = PySequence_Fast_ITEMS(o);
    for (Py_ssize_t i = 0; i < n; ++i) {
        long v;
        if (!read_int(items[i], &v)) return false;
        b->v[i] = (int32_t)v;
    }
    b->n = (int)n;
    return true;
}

// grid: None, or a pair (H, W)
bool read_grid(PyObject *o, bool *has, long *H, long *W)
{
    *has = o != Py_None;
    if (!*has) return true;
    if ((!PyTuple_Check(o) && !PyList_Check(o)) || PySequence_Fast_GET_SIZE(o) != 2) return false;
    return read_int(PySequence_Fast_GET_ITEM(o, 0), H) && read_int(PySequence_Fast_GET_ITEM(o, 1), W) && *H > 0 && *W > 0;
}

// No function transform, dispatch mode or trace is active on this thread.  Those act on torch's operators as they are called, and
// what happens here is none: left to the Python code, which they see (or which torch refuses under them).
bool plain_context()
{
    const c10::DispatchKeySet on = c10::impl::tls_local_dispatch_key_set().included_;
    return (on.raw_repr() & ~c10::default_included_set.raw_repr()) == 0;
}

// Dense device memory of its own: not a tensor that only stands for one (under a transform, a trace or a dispatch mode), nor
// one whose elements are to be read as something else (negated, zero).
bool usable(const at::Tensor &t)
{
    constexpr c10::DispatchKeySet plain({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::AutocastCUDA,
                                         c10::DispatchKey::ADInplaceOrView});
    return t.defined() && t.is_cuda() && t.layout() == at::kStrided && (t.key_set().raw_repr() & ~plain.raw_repr()) == 0;
}

// (subclasses of Tensor other than Parameter may override what is done with them)
// Undefined: an argument this module does not take.
at::Tensor read_tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return at::Tensor();
    const at::Tensor &t = THPVariable_Unpack(o);
    return usable(t) && t.is_contiguous() ? t : at::Tensor();
}

int dtype_code(at::ScalarType t) { return t == at::kFloat ? LBP_F32 : t == at::kBFloat16 ? LBP_BF16 : -1; }

bool small(int64_t v) { return v >= 0 && v <= INT32_MAX; }

bool read_stream(PyObject *o, c10::DeviceIndex dev, void **out)
{
    if (o == Py_None) {
        *out = (void *)c10::hip::getCurrentHIPStream(dev).stream();
        return true;
    }
    PyObject *p = PyObject_GetAttrString(o, "cuda_stream");
    if (!p) {
        PyErr_Clear();
        return false;
    }
    *out = PyLong_Check(p) ? PyLong_AsVoidPtr(p) : nullptr;
    const bool ok = PyLong_Check(p) && !PyErr_Occurred();
    Py_DECREF(p);
    PyErr_Clear();
    return ok;
}

// The caller's tensor for an output, if one was passed.  false: an argument this module does not take.
bool read_output(PyObject *o, at::IntArrayRef sizes, at::ScalarType dt, at::Device dev, at::Tensor *out)
{
    if (o == Py_None) return true;
    *out = read_tensor(o);
    return out->defined() && out->scalar_type() == dt && out->device() == dev && out->sizes() == sizes;
}

// A new output where one is wanted and the caller brought none.
void make_output(bool want, at::IntArrayRef sizes, at::ScalarType dt, at::Device dev, at::Tensor *out)
{
    if (want && !out->defined()) *out = at::detail::empty_cuda(sizes, at::TensorOptions().dtype(dt).device(dev));
}

void *address(const at::Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }

PyObject *wrap(const at::Tensor &t)
{
    if (!t.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(t);
}

PyObject *result(int rc, const at::Tensor &gx, const at::Tensor &gW)
{
    if (rc != LBP_OK) return PyLong_FromLong(rc);
    PyObject *a = wrap(gx), *b = wrap(gW), *tup = a && b ? PyTuple_New(2) : nullptr;
    if (!tup) {
        Py_XDECREF(a);
        Py_XDECREF(b);
        return nullptr;
    }
    PyTuple_SET_ITEM(tup, 0, a);
    PyTuple_SET_ITEM(tup, 1, b);
    return tup;
}

// The interpreter's lock is given up for the lifetime of this object.
class WithoutGil {
    PyThreadState *const state_ = PyEval_SaveThread();

public:
    WithoutGil() = default;
    WithoutGil(const WithoutGil &) = delete;
    WithoutGil &operator=(const WithoutGil &) = delete;
    ~WithoutGil() { PyEval_RestoreThread(state_); }
};

// backward(x, gy, w, grid, patch, basis_idx, gx, gW, want_gx, want_gw, gw_dtype, stream, kept)
// kept: x is x^, projected in the forward pass
PyObject *backward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 13 || !plain_context()) Py_RETURN_NONE;
    HANDLE_TH_ERRORS
    const at::Tensor x = read_tensor(a[0]), gy = read_tensor(a[1]), w = read_tensor(a[2]);
    bool has_grid;
    long H = 0, W = 0, patch;
    Bases idx;
    if (!x.defined() || !gy.defined() || !w.defined() || !read_grid(a[3], &has_grid, &H, &W) || !read_int(a[4], &patch) ||
        !read_bases(a[5], &idx) || !THPDtype_Check(a[10]))
        Py_RETURN_NONE;
    bool want_gx, want_gw, kept;
    if (!read_truth(a[8], &want_gx) || !read_truth(a[9], &want_gw) || !read_truth(a[12], &kept)) return nullptr;
    const at::ScalarType dt = x.scalar_type(), gw_dt = ((THPDtype *)a[10])->scalar_type;
    const at::Device dev = x.device();
    if (dtype_code(dt) < 0 || dtype_code(gw_dt) < 0 || gy.scalar_type() != dt || w.scalar_type() != dt ||
        gy.device() != dev || w.device() != dev || w.dim() != 2 || gy.dim() != (has_grid ? 3 : 4) || patch < 1)
        Py_RETURN_NONE;
    const int64_t N = gy.size(0), Cout = w.size(0), Cin = w.size(1);
    int64_t extra = 0;
    if (has_grid) {
        extra = gy.size(1) - (int64_t)H * W;
    } else {
        if (!small(gy.size(1)) || !small(gy.size(2))) Py_RETURN_NONE;
        H = gy.size(1);
        W = gy.size(2);
    }
    if (!small(N) || !small(Cin) || !small(Cout) || !small(extra) || gy.size(gy.dim() - 1) != Cout) Py_RETURN_NONE;
    int64_t gx_sizes[4] = {N, has_grid ? gy.size(1) : H, W, Cin};
    if (has_grid) gx_sizes[2] = Cin;
    const at::IntArrayRef gx_shape(gx_sizes, has_grid ? 3 : 4);
    if (kept) {
        const int64_t rows = N * ((H + patch - 1) / patch) * ((W + patch - 1) / patch) * idx.n + N * extra;
        if (x.dim() != 2 || x.size(0) != rows || x.size(1) != Cin) Py_RETURN_NONE;
    } else if (x.sizes() != gx_shape) {
        Py_RETURN_NONE;
    }
    void *stream;
    at::Tensor gx, gW;
    if (!read_stream(a[11], dev.index(), &stream) || !read_output(a[6], gx_shape, dt, dev, &gx) ||
        !read_output(a[7], w.sizes(), gw_dt, dev, &gW))
        Py_RETURN_NONE;
    const lbp_shape_t s = {(int32_t)N, (int32_t)H, (int32_t)W, (int32_t)Cin, (int32_t)Cout, dtype_code(dt), dtype_code(gw_dt)};
    int rc;
    {
        const WithoutGil unlocked;
        c10::OptionalDeviceGuard guard;
        guard.reset_device(dev);
        make_output(want_gx, gx_shape, dt, dev, &gx);
        make_output(want_gw, w.sizes(), gw_dt, dev, &gW);
        const auto call = kept ? lbp_wht_backward_tokens_preprojected : lbp_wht_backward_tokens;
        rc = call(x.data_ptr(), gy.data_ptr(), w.data_ptr(), &s, (int)extra, (int)patch, idx.v, idx.n, address(gx), address(gW), stream);
    }
    return result(rc, gx, gW);
    END_HANDLE_TH_ERRORS
}

// exact(x, gy, w, gx, gW, want_gx, want_gw, gw_dtype, stream)
PyObject *exact(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 9 || !plain_context()) Py_RETURN_NONE;
    HANDLE_TH_ERRORS
    const at::Tensor x = read_tensor(a[0]), gy = read_tensor(a[1]), w = read_tensor(a[2]);
    if (!x.defined() || !gy.defined() || !w.defined() || !THPDtype_Check(a[7]) || x.dim() != 4 || gy.dim() != 4 || w.dim() != 2)
        Py_RETURN_NONE;
    const at::ScalarType dt = x.scalar_type(), gw_dt = ((THPDtype *)a[7])->scalar_type;
    const at::Device dev = x.device();
    const int64_t N = x.size(0), H = x.size(1), W = x.size(2), Cin = x.size(3), Cout = gy.size(3);
    if (dtype_code(dt) < 0 || dtype_code(gw_dt) < 0 || gy.scalar_type() != dt || w.scalar_type() != dt ||
        gy.device() != dev || w.device() != dev || gy.size(0) != N || gy.size(1) != H || gy.size(2) != W ||
        w.size(0) != Cout || w.size(1) != Cin || !small(N) || !small(H) || !small(W) || !small(Cin) || !small(Cout))
        Py_RETURN_NONE;
    bool want_gx, want_gw;
    if (!read_truth(a[5], &want_gx) || !read_truth(a[6], &want_gw)) return nullptr;
    void *stream;
    at::Tensor gx, gW;
    if (!read_stream(a[8], dev.index(), &stream) || !read_output(a[3], x.sizes(), dt, dev, &gx) ||
        !read_output(a[4], w.sizes(), gw_dt, dev, &gW))
        Py_RETURN_NONE;
    const lbp_shape_t s = {(int32_t)N, (int32_t)H, (int32_t)W, (int32_t)Cin, (int32_t)Cout, dtype_code(dt), dtype_code(gw_dt)};
    int rc;
    {
        const WithoutGil unlocked;
        c10::OptionalDeviceGuard guard;
        guard.reset_device(dev);
        make_output(want_gx, x.sizes(), dt, dev, &gx);
        make_output(want_gw, w.sizes(), gw_dt, dev, &gW);
        rc = full_bp_backward(x.data_ptr(), gy.data_ptr(), w.data_ptr(), &s, address(gx), address(gW), stream);
    }
    return result(rc, gx, gW);
    END_HANDLE_TH_ERRORS
}

// The token grid of one tensor: [N,H,W,C], or [N,T,C] with grid = (H, W)
struct Grid {
    int64_t N, H, W, C, extra;
};

bool read_tokens(const at::Tensor &t, PyObject *grid, Grid *g)
{
    bool has;
    long H = 0, W = 0;
    if (!t.defined() || dtype_code(t.scalar_type()) < 0 || !read_grid(grid, &has, &H, &W) || t.dim() != (has ? 3 : 4)) return false;
    g->N = t.size(0);
    g->H = has ? H : t.size(1);
    g->W = has ? W : t.size(2);
    g->C = t.size(has ? 2 : 3);
    g->extra = has ? t.size(1) - g->H * g->W : 0;
    return small(g->N) && small(g->H) && small(g->W) && small(g->C) && small(g->extra);
}

// project(t, grid, patch, basis_idx, out, stream)
PyObject *project(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 6 || !plain_context()) Py_RETURN_NONE;
    HANDLE_TH_ERRORS
    const at::Tensor t = read_tensor(a[0]);
    Grid g;
    long patch;
    Bases idx;
    if (!read_tokens(t, a[1], &g) || !read_int(a[2], &patch) || patch < 1 || !read_bases(a[3], &idx)) Py_RETURN_NONE;
    const int64_t sizes[2] = {
        g.N * ((g.H + patch - 1) / patch) * ((g.W + patch - 1) / patch) * idx.n + g.N * g.extra, g.C};
    void *stream;
    at::Tensor out;
    if (!read_stream(a[5], t.device().index(), &stream) ||
        !read_output(a[4], at::IntArrayRef(sizes, 2), t.scalar_type(), t.device(), &out))
        Py_RETURN_NONE;
    int rc;
    {
        const WithoutGil unlocked;
        c10::OptionalDeviceGuard guard;
        guard.reset_device(t.device());
        make_output(true, at::IntArrayRef(sizes, 2), t.scalar_type(), t.device(), &out);
        rc = lbp_wht_project_tokens(t.data_ptr(), (int)g.N, (int)g.H, (int)g.W, (int)g.extra, (int)g.C, dtype_code(t.scalar_type()),
                                    (int)patch, idx.v, idx.n, out.data_ptr(), stream);
    }
    return rc == LBP_OK ? wrap(out) : PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// ---- the layer under autograd -------------------------------------------------------------------------------
//
// autograd.py's Function in native code: forward saves x^ and the weight only, backward is one call of the
// library with the bias gradient in it.  Of the 125 us of host time that a forward and backward pass of a small
// layer took in Python, most went through the two custom-function frames, their contexts and torch's reduction.

PyObject *error_class = nullptr;       // binding.py's LbpError

// Raises a status of the library as binding.py does; from any thread, without the interpreter's lock.
void raise_status(int rc)
{
    if (rc == LBP_OK) return;
    const int hip_error = lbp_last_hip_error();
    const PyGILState_STATE gil = PyGILState_Ensure();
    PyObject *error = error_class ? PyObject_CallFunction(error_class, "isi", rc, lbp_strerror(rc), hip_error) : nullptr;
    if (error) {
        PyErr_SetObject(error_class, error);
        Py_DECREF(error);
    } else if (!PyErr_Occurred()) {
        PyErr_SetString(PyExc_RuntimeError, lbp_strerror(rc));
    }
    python_error raised;
    raised.persist();       // (carries the exception to the thread that called backward)
    PyGILState_Release(gil);
    throw raised;
}

// use_error(LbpError)
PyObject *use_error(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n == 1 && PyExceptionClass_Check(a[0])) {
        Py_INCREF(a[0]);
        Py_XSETREF(error_class, a[0]);
    }
    Py_RETURN_NONE;
}

struct LbpWhtLinearBackward : public torch::autograd::Node {
    torch::autograd::SavedVariable x_r, weight;
    lbp_shape_t shape;
    int extra, patch;
    Bases idx;
    bool has_grid;
    c10::DeviceIndex device;

    // Saved-tensor hooks may hand back anything: what the kernels take by address is looked at as if a caller had passed it.
    void check_saved(const at::Tensor &xr, const at::Tensor &w) const
    {
        const at::Tensor *both[2] = {&xr, &w};
        for (const at::Tensor *t : both) {
            const char *name = t == &w ? "the saved weight" : "the saved x^";
            TORCH_CHECK_TYPE(usable(*t) && t->is_contiguous(), name, " must be a contiguous CUDA/HIP tensor");
            TORCH_CHECK_TYPE(dtype_code(t->scalar_type()) == shape.dtype, name, " must have the layer's dtype");
            TORCH_CHECK_VALUE(t->device().index() == device, name, " must be on the layer's device");
        }
        const int64_t patches = (int64_t)shape.N * ((shape.H + patch - 1) / patch) * ((shape.W + patch - 1) / patch);
        TORCH_CHECK_VALUE(xr.dim() == 2 && xr.size(0) == patches * idx.n + (int64_t)shape.N * extra && xr.size(1) == shape.Cin &&
                          w.dim() == 2 && w.size(0) == shape.Cout && w.size(1) == shape.Cin,
                          "the saved tensors must be x^ [P*r + N*extra, Cin] and the weight [Cout, Cin]");
    }

    torch::autograd::variable_list apply(torch::autograd::variable_list &&grads) override
    {
        std::lock_guard<std::mutex> lock(mutex_);
        const at::Tensor xr = x_r.unpack(), w = weight.unpack().detach();
        check_saved(xr, w);
        const at::Tensor &given = grads[0];
        at::Tensor gy = given.defined() ? given.detach().contiguous() : input_metadata(0).zeros_like();
        const bool want_x = task_should_compute_output(0), want_w = task_should_compute_output(1);
        const bool want_b = num_outputs() > 2 && task_should_compute_output(2);
        torch::autograd::variable_list out(num_outputs());
        TORCH_CHECK(usable(gy) && gy.device() == w.device(), "the output gradient must be a tensor on the layer's device");
        TORCH_CHECK_TYPE(gy.scalar_type() == w.scalar_type(), "the output gradient must have the layer's dtype");
        const int64_t N = shape.N, H = shape.H, W = shape.W, Cin = shape.Cin, Cout = shape.Cout;
        TORCH_CHECK_VALUE(has_grid ? gy.sizes() == at::IntArrayRef({N, extra + H * W, Cout}) : gy.sizes() == at::IntArrayRef({N, H, W, Cout}),
                          "the output gradient must have the output's shape");
        c10::OptionalDeviceGuard guard;
        guard.reset_device(w.device());
        const auto opts = at::TensorOptions().dtype(w.scalar_type()).device(w.device());
        if (want_x)
            out[0] = has_grid ? at::detail::empty_cuda({N, extra + H * W, Cin}, opts) : at::detail::empty_cuda({N, H, W, Cin}, opts);
        if (want_w) out[1] = at::detail::empty_cuda(w.sizes(), opts);
        // the bias gradient is linear in g_y: where somebody goes on from it (create_graph, a tangent on g_y), torch's own sum
        const bool sum_b = want_b && given.defined() &&
                           ((at::GradMode::is_enabled() && given.requires_grad()) || given._fw_grad(0).defined());
        if (sum_b) out[2] = given.sum(given.dim() == 3 ? at::IntArrayRef({0, 1}) : at::IntArrayRef({0, 1, 2}));
        else if (want_b) out[2] = at::detail::empty_cuda({Cout}, opts);
        void *gx = want_x ? out[0].data_ptr() : nullptr, *gW = want_w ? out[1].data_ptr() : nullptr;
        void *stream = (void *)c10::hip::getCurrentHIPStream(w.device().index()).stream();
        if (want_x || want_w) {
            if (want_b && !sum_b)
                raise_status(lbp_wht_backward_tokens_preprojected_bias(xr.data_ptr(), gy.data_ptr(), w.data_ptr(), &shape, extra, patch,
                                                                       idx.v, idx.n, gx, gW, out[2].data_ptr(), stream));
            else
                raise_status(lbp_wht_backward_tokens_preprojected(xr.data_ptr(), gy.data_ptr(), w.data_ptr(), &shape, extra, patch,
                                                                  idx.v, idx.n, gx, gW, stream));
        } else if (want_b && !sum_b) {
            out[2] = gy.reshape({-1, Cout}).sum(0);
        }
        return out;
    }

    void release_variables() override
    {
        std::lock_guard<std::mutex> lock(mutex_);
        x_r.reset_data();
        weight.reset_data();
    }

    std::string name() const override { return "LbpWhtLinearBackward"; }

    std::mutex &guard() { return mutex_; }
};

// grad_fn.saved_tensors, as on a Python Function
PyObject *saved_tensors(PyObject *self, void *)
{
    HANDLE_TH_ERRORS
    auto *node = static_cast<LbpWhtLinearBackward *>(((torch::autograd::THPCppFunction *)self)->cdata.get());
    at::Tensor x_r, weight;
    {
        const WithoutGil unlocked;      // (a backward pass on another thread may hold the node's lock and wait for the interpreter's)
        std::lock_guard<std::mutex> lock(node->guard());
        x_r = node->x_r.unpack();
        weight = node->weight.unpack();
    }
    PyObject *a = THPVariable_Wrap(x_r), *b = THPVariable_Wrap(weight);
    PyObject *tup = a && b ? PyTuple_New(2) : nullptr;
    if (!tup) {
        Py_XDECREF(a);
        Py_XDECREF(b);
        return nullptr;
    }
    PyTuple_SET_ITEM(tup, 0, a);
    PyTuple_SET_ITEM(tup, 1, b);
    return tup;
    END_HANDLE_TH_ERRORS
}

void register_node()
{
    using namespace torch::autograd;
    static PyTypeObject type;
    static PyGetSetDef props[] = {THP_FUNCTION_DEFAULT_PROPERTIES,
                                  {(char *)"saved_tensors", saved_tensors, nullptr, nullptr, nullptr},
                                  {nullptr, nullptr, nullptr, nullptr, nullptr}};
    static PyMethodDef node_methods[] = {{"_register_hook_dict", THPCppFunction_register_hook_dict, METH_O, nullptr},
                                         {"register_hook", THPCppFunction_register_hook, METH_O, nullptr},
                                         {"register_prehook", THPCppFunction_register_prehook, METH_O, nullptr},
                                         {"name", THPCppFunction_name, METH_NOARGS, nullptr},
                                         {"_sequence_nr", THPCppFunction_sequence_nr, METH_NOARGS, nullptr},
                                         {nullptr, nullptr, 0, nullptr}};
    if (_initFunctionPyTypeObject(type, "LbpWhtLinearBackward", props, node_methods)) {
        Py_INCREF(&type);
        registerCppFunction(typeid(LbpWhtLinearBackward), &type);
    }
}

// linear(x, weight, bias, grid, patch, basis_idx): y = x w^T (+ b) with the LBP-WHT backward
PyObject *linear(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 6 || !plain_context() || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    HANDLE_TH_ERRORS
    if (!THPVariable_CheckExact(a[0])) Py_RETURN_NONE;
    const at::Tensor x = THPVariable_Unpack(a[0]), w = read_tensor(a[1]);
    at::Tensor bias;
    bool has_grid;
    long H = 0, W = 0, patch;
    Bases idx;
    if (!usable(x) || !w.defined() || w.dim() != 2 || !read_grid(a[3], &has_grid, &H, &W) || !read_int(a[4], &patch) || patch < 1 ||
        !read_bases(a[5], &idx) || x.dim() != (has_grid ? 3 : 4))
        Py_RETURN_NONE;
    if (a[2] != Py_None && !(bias = read_tensor(a[2])).defined()) Py_RETURN_NONE;
    // forward-mode derivatives: torch refuses them for the Python function, which has none
    if (x._fw_grad(0).defined() || w._fw_grad(0).defined() || (bias.defined() && bias._fw_grad(0).defined())) Py_RETURN_NONE;
    const at::ScalarType dt = w.scalar_type();
    const at::Device dev = w.device();
    // (where autocast gives the product another type than the layer's)
    if (at::autocast::is_autocast_enabled(at::kCUDA) && at::autocast::get_autocast_dtype(at::kCUDA) != dt) Py_RETURN_NONE;
    const int64_t N = x.size(0), Cout = w.size(0), Cin = w.size(1);
    if (!has_grid) {
        if (!small(x.size(1)) || !small(x.size(2))) Py_RETURN_NONE;
        H = x.size(1);
        W = x.size(2);
    }
    const int64_t extra = has_grid ? x.size(1) - (int64_t)H * W : 0;
    if (dtype_code(dt) < 0 || x.scalar_type() != dt || x.device() != dev || x.size(x.dim() - 1) != Cin || !small(N) || !small(Cin) ||
        !small(Cout) || !small(extra) || (bias.defined() && (bias.scalar_type() != dt || bias.device() != dev || bias.dim() != 1 ||
        bias.size(0) != Cout)))
        Py_RETURN_NONE;
    at::Tensor y, x_r;
    int rc;
    {
        const WithoutGil unlocked;
        at::NoGradGuard no_grad;
        c10::OptionalDeviceGuard guard;
        guard.reset_device(dev);
        const at::Tensor xc = x.detach().contiguous();
        y = at::linear(xc, w.detach(), bias.defined() ? c10::optional<at::Tensor>(bias.detach()) : c10::nullopt);
        const int64_t rows = N * ((H + patch - 1) / patch) * ((W + patch - 1) / patch) * idx.n + N * extra;
        x_r = at::detail::empty_cuda({rows, Cin}, at::TensorOptions().dtype(dt).device(dev));
        rc = lbp_wht_project_tokens(xc.data_ptr(), (int)N, (int)H, (int)W, (int)extra, (int)Cin, dtype_code(dt), (int)patch,
                                    idx.v, idx.n, x_r.data_ptr(), (void *)c10::hip::getCurrentHIPStream(dev.index()).stream());
    }
    if (rc != LBP_OK) return PyLong_FromLong(rc);
    const bool needed = at::GradMode::is_enabled() && (x.requires_grad() || w.requires_grad() || (bias.defined() && bias.requires_grad()));
    if (needed) {
        auto node = std::shared_ptr<LbpWhtLinearBackward>(new LbpWhtLinearBackward(), torch::autograd::deleteNode);
        node->set_next_edges(bias.defined() ? torch::autograd::collect_next_edges(x, w, bias) : torch::autograd::collect_next_edges(x, w));
        node->x_r = torch::autograd::SavedVariable(x_r, false);
        node->weight = torch::autograd::SavedVariable(w, false);
        node->shape = lbp_shape_t{(int32_t)N, (int32_t)H, (int32_t)W, (int32_t)Cin, (int32_t)Cout, dtype_code(dt), dtype_code(dt)};
        node->extra = (int)extra;
        node->patch = (int)patch;
        node->idx = idx;
        node->has_grid = has_grid;
        node->device = dev.index();
        torch::autograd::set_history(y, node);
    }
    return wrap(y);
    END_HANDLE_TH_ERRORS
}

// energy(t, grid, patch, energy, stream)
PyObject *energy(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 5 || !plain_context()) Py_RETURN_NONE;
    HANDLE_TH_ERRORS
    const at::Tensor t = read_tensor(a[0]);
    Grid g;
    long patch;
    if (!read_tokens(t, a[1], &g) || !read_int(a[2], &patch) || patch < 1 || patch > 16) Py_RETURN_NONE;
    const int64_t bases = (int64_t)patch * patch;
    void *stream;
    at::Tensor e;
    const bool fresh = a[3] == Py_None;      // a new spectrum is written, the caller's is added to
    if (!read_stream(a[4], t.device().index(), &stream) ||
        !read_output(a[3], at::IntArrayRef(&bases, 1), at::kDouble, t.device(), &e))
        Py_RETURN_NONE;
    int rc;
    {
        const WithoutGil unlocked;
        c10::OptionalDeviceGuard guard;
        guard.reset_device(t.device());
        make_output(true, at::IntArrayRef(&bases, 1), at::kDouble, t.device(), &e);
        const auto call = fresh ? lbp_wht_energy_tokens_overwrite : lbp_wht_energy_tokens;
        rc = call(t.data_ptr(), (int)g.N, (int)g.H, (int)g.W, (int)g.extra, (int)g.C, dtype_code(t.scalar_type()), (int)patch,
                  (double *)e.data_ptr(), stream);
    }
    return rc == LBP_OK ? wrap(e) : PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

#define LBP_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {LBP_METHOD(backward), LBP_METHOD(exact), LBP_METHOD(project), LBP_METHOD(linear),
                         LBP_METHOD(energy), LBP_METHOD(use_error),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    PyObject *m = PyModule_Create(&module);
    if (m) register_node();
    return m;
}
