// The one-call convenience function on torch tensors, natively: what conv_fwd_fused of the Python binding does for plain
// arguments, without the interpreter.  A tiny layer's launch takes the GPU about 3.6 us and took the host 8 in Python and
// ctypes.  Anything out of the ordinary (tensor subclasses and wrappers, other argument types, options, errors) is left to the
// Python function: this one then returns None and has done nothing.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/cvx.h"

namespace {

// A thread's handles (one a device) and descriptors; the descriptors are set by each call, and a handle keeps the
// plans of the problems it met last.  Closed when the thread ends.
struct Thread {
    static constexpr int DEVICES = 16;
    cvx_handle_t handle[DEVICES] = {};
    cvx_tensor_desc_t x = nullptr, w = nullptr, y = nullptr, b = nullptr;
    cvx_conv_desc_t conv = nullptr;

    bool ready(int device)
    {
        if (device < 0 || device >= DEVICES) return false;
        if (!conv && (cvx_tensor_desc_create(&x) || cvx_tensor_desc_create(&w) || cvx_tensor_desc_create(&y) || cvx_tensor_desc_create(&b) ||
                      cvx_conv_desc_create(&conv)))
            return false;
        return handle[device] || cvx_create(&handle[device], nullptr) == CVX_OK;
    }
    ~Thread()
    {
        for (cvx_handle_t h : handle)
            if (h) cvx_destroy(h);
        for (cvx_tensor_desc_t t : {x, w, y, b})
            if (t) cvx_tensor_desc_destroy(t);
        if (conv) cvx_conv_desc_destroy(conv);
    }
};

bool dtype_code(const at::Tensor& t, cvx_dtype_t* out)
{
    switch (t.scalar_type()) {
    case at::kFloat: *out = CVX_F32; return true;
    case at::kHalf: *out = CVX_F16; return true;
    case at::kBFloat16: *out = CVX_BF16; return true;
    default: return false;
    }
}

// A dense GPU tensor with memory of its own behind it: no subclass, no wrapper of a transform or a mode, no lazy
// conjugate or negative.
bool plain(PyObject* o, const at::Tensor** out)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    const c10::DispatchKeySet extra = t.key_set() - c10::autograd_dispatch_keyset - c10::autocast_dispatch_keyset - c10::DispatchKeySet(c10::DispatchKey::ADInplaceOrView);
    *out = &t;
    return extra == c10::DispatchKeySet(c10::DispatchKey::CUDA) && t.is_contiguous();
}

bool whole(PyObject* o, int* out)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    *out = (int)v;
    return !over && v == (long)*out;
}

bool pair(PyObject* o, int* h, int* w)
{
    if (whole(o, h)) {
        *w = *h;
        return true;
    }
    return PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) >= 2 && whole(PyTuple_GET_ITEM(o, 0), h) && whole(PyTuple_GET_ITEM(o, 1), w);
}

bool dims(const at::Tensor& t, int (&d)[4])
{
    if (t.dim() != 4) return false;
    for (int i = 0; i < 4; ++i) {
        if (t.size(i) < 1 || t.size(i) > 0x7fffffff) return false;
        d[i] = (int)t.size(i);
    }
    return true;
}

PyObject* none() { Py_RETURN_NONE; }

// (x, w, bias, pad, stride, dil, groups, act, alpha) -> y, or None: the caller goes the long way
PyObject* conv_fwd_fused(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != 9) return none();
    const at::Tensor *x, *w, *b = nullptr;
    cvx_dtype_t dt, wdt, bdt = CVX_F32;
    int xd[4], wd[4], ph, pw, sh, sw, dh, dw, groups, act;
    if (!plain(args[0], &x) || !plain(args[1], &w) || !dtype_code(*x, &dt) || !dtype_code(*w, &wdt) || wdt != dt || !dims(*x, xd) || !dims(*w, wd)) return none();
    if (args[2] != Py_None && (!plain(args[2], &b) || !dtype_code(*b, &bdt) || b->numel() != wd[0])) return none();
    if (!pair(args[3], &ph, &pw) || !pair(args[4], &sh, &sw) || !pair(args[5], &dh, &dw) || !whole(args[6], &groups) || !whole(args[7], &act)) return none();
    if (act < CVX_ACT_IDENTITY || act > CVX_ACT_LOGISTIC || !PyFloat_CheckExact(args[8])) return none();
    const c10::impl::LocalDispatchKeySet tls = c10::impl::tls_local_dispatch_key_set();
    if (tls.included_.has_any(c10::python_ks | c10::functorch_transforms_ks)) return none();
    const int device = x->get_device();
    if (w->get_device() != device || (b && b->get_device() != device)) return none();

    static thread_local Thread mine;
    int yn, yk, yh, yw;
    if (!mine.ready(device) || cvx_tensor_desc_set_4d(mine.x, dt, xd[0], xd[1], xd[2], xd[3]) || cvx_tensor_desc_set_4d(mine.w, dt, wd[0], wd[1], wd[2], wd[3]) ||
        cvx_conv_desc_set_2d(mine.conv, ph, pw, sh, sw, dh, dw) || cvx_conv_desc_set_group_count(mine.conv, groups) ||
        cvx_conv_fwd_output_dim(mine.conv, mine.x, mine.w, &yn, &yk, &yh, &yw) || cvx_tensor_desc_set_4d(mine.y, dt, yn, yk, yh, yw) ||
        (b && cvx_tensor_desc_set_4d(mine.b, bdt, 1, yk, 1, 1)))
        return none();
    try {
        at::Tensor y = at::empty({yn, yk, yh, yw}, at::TensorOptions().dtype(x->scalar_type()).device(x->device()));
        cvx_set_stream(mine.handle[device], (void*)c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream());
        const float alpha = (float)PyFloat_AS_DOUBLE(args[8]);
        cvx_status_t st;
        const void *xp = x->const_data_ptr(), *wp = w->const_data_ptr(), *bp = b ? b->const_data_ptr() : nullptr;
        void* yp = y.mutable_data_ptr();
        Py_BEGIN_ALLOW_THREADS
        st = cvx_conv_fwd_fused(mine.handle[device], mine.x, xp, mine.w, wp, mine.conv, b ? mine.b : nullptr, bp, (cvx_act_t)act, alpha, mine.y, yp);
        Py_END_ALLOW_THREADS
        if (st != CVX_OK) return none();
        return THPVariable_Wrap(std::move(y));
    } catch (const std::exception&) {
        return none();                                   // out of memory and the like: the long way raises it
    }
}

PyMethodDef methods[] = {{"conv_fwd_fused", (PyCFunction)(void (*)(void))conv_fwd_fused, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_cvx_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__cvx_torch()
{
    PyObject* const m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", CVX_TORCH_VERSION) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
