// Host path of the layers (layer.py): one call per autograd step that lays out the tensors, allocates outputs, state and
// scratch with torch's allocator and enqueues the library's kernels through its C ABI.  Done in Python the same steps cost
// several times as long as the kernels of a small layer (C1, forward and backward: 230 us of host time for 60 us of kernels).
// No arithmetic here.  The library's functions are looked up in the very library that binding.py has loaded.
#include <Python.h>
#include <dlfcn.h>

#include <ATen/ATen.h>
#include <c10/core/DeviceGuard.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <string>

#include "../../include/xconv.h"

namespace {

using at::Tensor;

struct Lib {
    decltype(&xconv_check_desc) check_desc;
    decltype(&xconv_xt_bytes) xt_bytes;
    decltype(&xconv_workspace_bytes) workspace_bytes;
    decltype(&xconv_conv_workspace_bytes) conv_workspace_bytes;
    decltype(&xconv_conv_fwd_ws) conv_fwd;
    decltype(&xconv_dx_exact_ws) dx_exact;
    decltype(&xconv_probe_fwd) probe_fwd;
    decltype(&xconv_dw_estimate_as) dw_estimate;
    decltype(&xconv_bias_workspace_bytes) bias_workspace_bytes;
    decltype(&xconv_bias_grad) bias_grad;
    decltype(&xconv_pixel_xbar_bytes) pixel_xbar_bytes, indep_xbar_bytes;
    decltype(&xconv_pixel_workspace_bytes) pixel_workspace_bytes, indep_workspace_bytes;
    decltype(&xconv_pixel_probe_fwd) pixel_probe_fwd, indep_probe_fwd;
    decltype(&xconv_pixel_dw_estimate_as) pixel_dw_estimate;
    decltype(&xconv_pixel_indep_dw_estimate) indep_dw_estimate;
    decltype(&xconv_layer_workspace_bytes) layer_workspace_bytes;
    decltype(&xconv_layer_fwd) layer_fwd;
    decltype(&xconv_layer_bwd) layer_bwd;
    decltype(&xconv_relu_mask_bytes) relu_mask_bytes;
    decltype(&xconv_relu_fwd) relu_fwd;
    decltype(&xconv_relu_bwd) relu_bwd;
    decltype(&xconv_status_string) status_string;
} L;
bool g_ready = false;

enum Mode { kChannel = 0, kMulti = 1, kIndependent = 2 };

struct Failed {   // a status of the library
    int status;
    const char *where;
};
void check(xconv_status s, const char *where)
{
    if (s != XCONV_OK) throw Failed{(int)s, where};
}
PyObject *g_error_type = nullptr;   // binding.XConvError(status, where)

int dtype_code(at::ScalarType t)
{
    return t == at::kFloat ? XCONV_F32 : t == at::kBFloat16 ? XCONV_BF16 : XCONV_F16;
}
bool aligned16(const Tensor &t) { return (reinterpret_cast<uintptr_t>(t.data_ptr()) & 15u) == 0; }
// the library takes 16-byte aligned tensors; a view into the middle of a storage may not be
Tensor aligned(const Tensor &t) { return aligned16(t) ? t : t.clone(at::MemoryFormat::Preserve); }
// (layout code, tensor whose memory is in that layout)
Tensor in_layout(const Tensor &x, int &layout)
{
    layout = XCONV_NCHW;
    if (x.is_contiguous()) return aligned(x);
    if (x.is_contiguous(at::MemoryFormat::ChannelsLast)) {
        layout = XCONV_NHWC;
        return aligned(x);
    }
    return x.contiguous();
}
at::MemoryFormat format_of(int layout) { return layout == XCONV_NHWC ? at::MemoryFormat::ChannelsLast : at::MemoryFormat::Contiguous; }
Tensor bytes_on(size_t n, const Tensor &like)
{
    return at::empty({(int64_t)(n < 16 ? 16 : n)}, like.options().dtype(at::kByte));
}
void *ptr(const Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }

[[noreturn]] void unsupported(const xconv_desc &d)
{
    throw std::runtime_error("XConv2d: layer not supported by the library in this mode (C_in=" + std::to_string(d.C_in) + ", " + std::to_string(d.H) + "x" +
                             std::to_string(d.W) + ", r=" + std::to_string(d.r) + ")");
}

// One Python call: runs `body` without the interpreter lock, turns failures into Python errors: a status of the library into
// XConvError, everything else into what torch makes of it (torch.OutOfMemoryError for an allocation, say)
template <class F> bool run(F &&body)
{
    std::exception_ptr other;
    int status = -1;
    const char *where = "";
    Py_BEGIN_ALLOW_THREADS
    try {
        at::AutoDispatchBelowADInplaceOrView below;
        body();
        status = 0;
    } catch (const Failed &f) {
        status = f.status;
        where = f.where;
    } catch (...) {
        other = std::current_exception();
    }
    Py_END_ALLOW_THREADS
    if (status == 0) return true;
    if (status > 0) {
        PyObject *e = PyObject_CallFunction(g_error_type, "is", status, where);
        if (e) {
            PyErr_SetObject(g_error_type, e);
            Py_DECREF(e);
        }
    } else {
        torch::translate_exception_to_python(other);
    }
    return false;
}

Tensor tensor_arg(PyObject *o) { return o == Py_None ? Tensor() : THPVariable_Unpack(o); }
PyObject *wrap(const Tensor &t)
{
    if (!t.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(t);
}
bool ints(PyObject *const *args, int first, int n, long long *out)
{
    for (int i = 0; i < n; ++i) {
        out[i] = PyLong_AsLongLong(args[first + i]);
        if (out[i] == -1 && PyErr_Occurred()) return false;
    }
    return true;
}
bool ready(Py_ssize_t n, Py_ssize_t want, const char *name)
{
    if (!g_ready) {
        PyErr_SetString(PyExc_RuntimeError, "torch glue: init() has not been called");
        return false;
    }
    if (n != want) {
        PyErr_Format(PyExc_TypeError, "%s: %zd arguments, %zd expected", name, n, want);
        return false;
    }
    return true;
}

// forward(x, weight, bias, stride_h, stride_w, pad_h, pad_w, r, probe, mode, seed, own, state, stream)
//   -> (y or None, state or None, desc bytes)
PyObject *layer_forward(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (!ready(nargs, 14, "forward")) return nullptr;
    const Tensor x = tensor_arg(args[0]), weight = tensor_arg(args[1]), bias = tensor_arg(args[2]);
    long long v[11];
    if (!ints(args, 3, 11, v)) return nullptr;
    const int mode = (int)v[6];
    const bool own = v[8] != 0, want_state = v[9] != 0;
    void *stream = reinterpret_cast<void *>(v[10]);
    xconv_desc d{};
    Tensor y, state;
    if (!run([&] {
            const c10::DeviceGuard guard(x.device());
            // the kernels take the weight's extents from the descriptor
            if (x.dim() != 4 || weight.dim() != 4 || x.size(1) != weight.size(1))
                throw std::runtime_error("XConv2d: expected an input of 4 dimensions with " + std::to_string(weight.size(1)) + " channels");
            int layout;
            const Tensor xs = in_layout(x, layout);
            d.B = (int)x.size(0); d.C_in = (int)x.size(1); d.H = (int)x.size(2); d.W = (int)x.size(3);
            d.C_out = (int)weight.size(0); d.kH = (int)weight.size(2); d.kW = (int)weight.size(3);
            d.stride_h = (int)v[0]; d.stride_w = (int)v[1]; d.pad_h = (int)v[2]; d.pad_w = (int)v[3];
            d.r = (int)v[4]; d.probe = (int)v[5]; d.dtype = dtype_code(x.scalar_type()); d.layout = layout;
            d.seed = (uint64_t)v[7];
            // before anything is computed from it (a stride of 0, an empty output); what the library does not support is reported below
            if (L.check_desc(&d) == XCONV_EINVAL) throw Failed{XCONV_EINVAL, "xconv_check_desc"};
            Tensor w, b;
            // the kernel reads one bias per output channel in the storage type; any other bias (a float32 one of a half-precision
            // layer, say) is added behind it
            const bool apart = own && bias.defined() &&
                               (bias.scalar_type() != x.scalar_type() || bias.device() != x.device() || bias.dim() != 1 || bias.size(0) != weight.size(0));
            auto add_apart = [&] {
                if (apart) y.add_(bias.view({1, -1, 1, 1}));
            };
            if (own) {
                w = weight.contiguous();
                if (bias.defined() && !apart) b = bias.contiguous();
                const int64_t Ho = (d.H + 2 * d.pad_h - d.kH) / d.stride_h + 1, Wo = (d.W + 2 * d.pad_w - d.kW) / d.stride_w + 1;
                y = at::empty({d.B, d.C_out, Ho, Wo}, x.options(), format_of(layout));
            }
            if (want_state) {
                const size_t n = mode == kChannel ? L.xt_bytes(&d) : (mode == kIndependent ? L.indep_xbar_bytes : L.pixel_xbar_bytes)(&d);
                if (n == 0) unsupported(d);
                state = mode == kChannel ? bytes_on(n, x) : at::empty({(int64_t)(n / 4)}, x.options().dtype(at::kFloat));
            }
            if (own && want_state && mode != kIndependent) {
                const size_t n = L.layer_workspace_bytes(&d, mode, 0);
                if (n == 0 || (mode == kChannel && L.workspace_bytes(&d, XCONV_OP_ESTIMATE) == 0)) unsupported(d);
                const Tensor ws = bytes_on(n, x);
                check(L.layer_fwd(&d, mode, ptr(xs), ptr(w), ptr(b), ptr(y), ptr(state), ptr(ws), (size_t)ws.numel(), stream), "xconv_layer_fwd");
                add_apart();
                return;
            }
            if (own) {
                const Tensor ws = bytes_on(L.conv_workspace_bytes(&d, 0), x);
                check(L.conv_fwd(&d, ptr(xs), ptr(w), ptr(b), ptr(y), ptr(ws), (size_t)ws.numel(), stream), "xconv_conv_fwd_ws");
                add_apart();
            }
            if (!want_state) return;
            if (mode == kChannel) {
                const size_t n = L.workspace_bytes(&d, XCONV_OP_PROBE);
                if (L.workspace_bytes(&d, XCONV_OP_ESTIMATE) == 0) unsupported(d);
                const Tensor ws = bytes_on(n, x);
                check(L.probe_fwd(&d, ptr(xs), ptr(state), nullptr, ptr(ws), (size_t)ws.numel(), stream), "xconv_probe_fwd");
            } else {
                const bool indep = mode == kIndependent;
                const size_t n = (indep ? L.indep_workspace_bytes : L.pixel_workspace_bytes)(&d, XCONV_OP_PROBE);
                if (n == 0) unsupported(d);
                const Tensor ws = bytes_on(n, x);
                check((indep ? L.indep_probe_fwd : L.pixel_probe_fwd)(&d, ptr(xs), state.data_ptr<float>(), ptr(ws), (size_t)ws.numel(), stream),
                      "xconv_pixel_probe_fwd");
            }
        }))
        return nullptr;
    return Py_BuildValue("NNy#", wrap(y), wrap(state), reinterpret_cast<const char *>(&d), (Py_ssize_t)sizeof(d));
}

// backward(dy, weight, state or None, desc bytes, mode, need_dx, need_dw, need_db, stream) -> (dx, dw, db), None where not asked for
PyObject *layer_backward(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (!ready(nargs, 9, "backward")) return nullptr;
    const Tensor dy = tensor_arg(args[0]), weight = tensor_arg(args[1]), state = tensor_arg(args[2]);
    char *raw;
    Py_ssize_t len;
    if (PyBytes_AsStringAndSize(args[3], &raw, &len) < 0) return nullptr;
    if (len != (Py_ssize_t)sizeof(xconv_desc)) {
        PyErr_SetString(PyExc_ValueError, "backward: not a descriptor");
        return nullptr;
    }
    xconv_desc d;
    memcpy(&d, raw, sizeof(d));
    long long v[5];
    if (!ints(args, 4, 5, v)) return nullptr;
    const int mode = (int)v[0];
    void *stream = reinterpret_cast<void *>(v[4]);
    Tensor dx, dw, db;
    if (!run([&] {
            const c10::DeviceGuard guard(dy.device());
            const at::ScalarType xt = d.dtype == XCONV_F32 ? at::kFloat : d.dtype == XCONV_BF16 ? at::kBFloat16 : at::kHalf;
            int layout;
            Tensor dys = in_layout(dy, layout);
            // the gradient comes in the weight's type where that is a storage type (independent probing adds up fp32 pieces first)
            const at::ScalarType wst = weight.scalar_type();
            const bool direct = mode != kIndependent && (wst == at::kFloat || wst == at::kBFloat16 || wst == at::kHalf);
            if (v[2] && direct && layout == d.layout && dys.scalar_type() == xt) {
                const Tensor w = v[1] ? weight.contiguous() : weight;
                if (v[1]) dx = at::empty({d.B, d.C_in, d.H, d.W}, dy.options(), format_of(layout));
                if (v[3]) db = at::empty({d.C_out}, dy.options());
                dw = at::empty(weight.sizes(), weight.options(), at::MemoryFormat::Contiguous);
                const Tensor ws = bytes_on(L.layer_workspace_bytes(&d, mode, 1), dy);
                check(L.layer_bwd(&d, mode, ptr(dys), ptr(w), ptr(state), ptr(dx), ptr(dw), dtype_code(wst), ptr(db), ptr(ws), (size_t)ws.numel(), stream),
                      "xconv_layer_bwd");
                return;
            }
            if (v[1]) {
                xconv_desc q = d;
                q.layout = layout;
                q.dtype = dtype_code(dy.scalar_type());
                const Tensor w = weight.contiguous();
                dx = at::empty({d.B, d.C_in, d.H, d.W}, dy.options(), format_of(layout));
                const Tensor ws = bytes_on(L.conv_workspace_bytes(&q, 1), dy);
                check(L.dx_exact(&q, ptr(dys), ptr(w), ptr(dx), ptr(ws), (size_t)ws.numel(), stream), "xconv_dx_exact_ws");
            }
            if (v[3]) {
                xconv_desc q = d;
                q.layout = layout;
                q.dtype = dtype_code(dy.scalar_type());
                db = at::empty({d.C_out}, dy.options());
                const Tensor ws = bytes_on(L.bias_workspace_bytes(&q), dy);
                check(L.bias_grad(&q, ptr(dys), ptr(db), ptr(ws), (size_t)ws.numel(), stream), "xconv_bias_grad");
            }
            if (v[2]) {
                if (dys.scalar_type() != xt) {
                    dys = dys.to(xt);
                    if (!aligned16(dys)) dys = dys.clone(at::MemoryFormat::Preserve);
                }
                if (layout != d.layout) dys = aligned(dys.contiguous(format_of(d.layout)));
                const bool indep = mode == kIndependent;
                dw = at::empty(weight.sizes(), weight.options().dtype(direct ? wst : at::kFloat), at::MemoryFormat::Contiguous);
                const int wt = dtype_code(dw.scalar_type());
                const size_t n = mode == kChannel ? L.workspace_bytes(&d, XCONV_OP_ESTIMATE)
                                                  : (indep ? L.indep_workspace_bytes : L.pixel_workspace_bytes)(&d, XCONV_OP_ESTIMATE);
                const Tensor ws = bytes_on(n, dy);
                if (mode == kChannel)
                    check(L.dw_estimate(&d, ptr(dys), ptr(state), nullptr, ptr(dw), wt, ptr(ws), (size_t)ws.numel(), stream), "xconv_dw_estimate_as");
                else if (!indep)
                    check(L.pixel_dw_estimate(&d, ptr(dys), state.data_ptr<float>(), ptr(dw), wt, ptr(ws), (size_t)ws.numel(), stream),
                          "xconv_pixel_dw_estimate_as");
                else
                    check(L.indep_dw_estimate(&d, ptr(dys), state.data_ptr<float>(), dw.data_ptr<float>(), ptr(ws), (size_t)ws.numel(), stream),
                          "xconv_pixel_indep_dw_estimate");
                if (!direct) dw = dw.to(wst);
            }
        }))
        return nullptr;
    return Py_BuildValue("NNN", wrap(dx), wrap(dw), wrap(db));
}

// relu_forward(x, stream) -> (y, mask)
PyObject *relu_forward(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (!ready(nargs, 2, "relu_forward")) return nullptr;
    const Tensor x = tensor_arg(args[0]);
    long long s;
    if (!ints(args, 1, 1, &s)) return nullptr;
    Tensor y, mask;
    if (!run([&] {
            const c10::DeviceGuard guard(x.device());
            // values in memory order: the mask is per element, whatever the layout
            Tensor xs = x;
            if (!(x.is_contiguous() || x.is_contiguous(at::MemoryFormat::ChannelsLast) || (x.dim() == 5 && x.is_contiguous(at::MemoryFormat::ChannelsLast3d))))
                xs = x.contiguous();
            xs = aligned(xs);
            y = at::empty_like(xs);     // same strides as xs
            const int64_t n = xs.numel();
            mask = at::empty({std::max<int64_t>((int64_t)L.relu_mask_bytes(n) / 8, 1)}, x.options().dtype(at::kLong));
            check(L.relu_fwd(dtype_code(x.scalar_type()), ptr(xs), ptr(y), ptr(mask), n, reinterpret_cast<void *>(s)), "xconv_relu_fwd");
        }))
        return nullptr;
    return Py_BuildValue("NN", wrap(y), wrap(mask));
}

// relu_backward(dy, mask, shape, strides, dtype code, stream) -> dx; the gradient in the memory order of the output
PyObject *relu_backward(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (!ready(nargs, 6, "relu_backward")) return nullptr;
    const Tensor dy = tensor_arg(args[0]), mask = tensor_arg(args[1]);
    std::vector<int64_t> dims[2];
    for (int k = 0; k < 2; ++k)
        for (Py_ssize_t i = 0; i < PyTuple_Size(args[2 + k]); ++i) dims[k].push_back(PyLong_AsLongLong(PyTuple_GetItem(args[2 + k], i)));
    long long v[2];
    if (PyErr_Occurred() || !ints(args, 4, 2, v)) return nullptr;
    Tensor dx;
    if (!run([&] {
            const c10::DeviceGuard guard(dy.device());
            const at::ScalarType t = v[0] == XCONV_F32 ? at::kFloat : v[0] == XCONV_BF16 ? at::kBFloat16 : at::kHalf;
            dx = at::empty_strided(dims[0], dims[1], dy.options().dtype(t));
            Tensor src = dy;
            // a gradient that already lies in that order is read where it is
            if (dy.scalar_type() != t || dy.sizes() != dx.sizes() || dy.strides() != dx.strides() || !aligned16(dy)) {
                dx.copy_(dy);
                src = dx;
            }
            check(L.relu_bwd((int)v[0], ptr(src), ptr(mask), ptr(dx), dx.numel(), reinterpret_cast<void *>(v[1])), "xconv_relu_bwd");
        }))
        return nullptr;
    return wrap(dx);
}

// init(path of the loaded library, error type)
PyObject *glue_init(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (nargs != 2) {
        PyErr_SetString(PyExc_TypeError, "init: 2 arguments expected");
        return nullptr;
    }
    const char *path = PyUnicode_AsUTF8(args[0]);
    if (!path) return nullptr;
    void *h = dlopen(path, RTLD_NOW);
    if (!h) {
        PyErr_SetString(PyExc_RuntimeError, dlerror());
        return nullptr;
    }
    const char *missing = nullptr;
    auto get = [&](auto &f, const char *name) {
        f = reinterpret_cast<std::remove_reference_t<decltype(f)>>(dlsym(h, name));
        if (!f) missing = name;
    };
    get(L.check_desc, "xconv_check_desc");
    get(L.xt_bytes, "xconv_xt_bytes");
    get(L.workspace_bytes, "xconv_workspace_bytes");
    get(L.conv_workspace_bytes, "xconv_conv_workspace_bytes");
    get(L.conv_fwd, "xconv_conv_fwd_ws");
    get(L.dx_exact, "xconv_dx_exact_ws");
    get(L.probe_fwd, "xconv_probe_fwd");
    get(L.dw_estimate, "xconv_dw_estimate_as");
    get(L.bias_workspace_bytes, "xconv_bias_workspace_bytes");
    get(L.bias_grad, "xconv_bias_grad");
    get(L.pixel_xbar_bytes, "xconv_pixel_xbar_bytes");
    get(L.indep_xbar_bytes, "xconv_pixel_indep_xbar_bytes");
    get(L.pixel_workspace_bytes, "xconv_pixel_workspace_bytes");
    get(L.indep_workspace_bytes, "xconv_pixel_indep_workspace_bytes");
    get(L.pixel_probe_fwd, "xconv_pixel_probe_fwd");
    get(L.indep_probe_fwd, "xconv_pixel_indep_probe_fwd");
    get(L.pixel_dw_estimate, "xconv_pixel_dw_estimate_as");
    get(L.indep_dw_estimate, "xconv_pixel_indep_dw_estimate");
    get(L.layer_workspace_bytes, "xconv_layer_workspace_bytes");
    get(L.layer_fwd, "xconv_layer_fwd");
    get(L.layer_bwd, "xconv_layer_bwd");
    get(L.relu_mask_bytes, "xconv_relu_mask_bytes");
    get(L.relu_fwd, "xconv_relu_fwd");
    get(L.relu_bwd, "xconv_relu_bwd");
    get(L.status_string, "xconv_status_string");
    if (missing) {
        PyErr_Format(PyExc_RuntimeError, "%s has no %s", path, missing);
        return nullptr;
    }
    Py_XDECREF(g_error_type);
    Py_INCREF(args[1]);
    g_error_type = args[1];
    g_ready = true;
    Py_RETURN_NONE;
}

#define XC_METHOD(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(fn)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    XC_METHOD("init", glue_init),
    XC_METHOD("forward", layer_forward),
    XC_METHOD("backward", layer_backward),
    XC_METHOD("relu_forward", relu_forward),
    XC_METHOD("relu_backward", relu_backward),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_torch_glue", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_glue(void) { return PyModule_Create(&g_module); }
