// The single-layer calls of binding.py without Python in between: argument checks, the output tensors and
// the C-ABI call.  A call of a small layer is bound by its host side: of 6.5 us the launch takes 3.4, and in
// Python the output tensor took 1.5, marshalling 0.6, the checks 0.5 and the stream 0.2; here all of these take 1.3
// (a 64->64 layer at 64x64 6.6 -> 4.3 to 4.8 us, the other small calls 6.1-7.2 -> 4.8-5.1).
//
// Every function takes the plain case only - tensors of the exact type, on the device, contiguous, of the
// expected dtype, no function or dispatch mode active - and returns None for anything else, so that the general
// code in binding.py decides (and raises) as it does.  Otherwise it returns the outputs, or the C-ABI's error code.
#include <Python.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/device_lazy_init.h>
#include "mbu.h"

namespace {

// addresses of the loaded C-ABI library, and torch's accessors of the current device and its current stream
struct {
    decltype(&mbu_conv3x3_masked_binary) conv;
    decltype(&mbu_conv3x3_masked_binary_fused) fused;
    decltype(&mbu_conv3x3_masked_binary_concat) concat;
    decltype(&mbu_conv3x3_masked_binary_two_inputs) two;
    decltype(&mbu_tconv2x2_masked_binary) tconv;
    decltype(&mbu_pack_act) pack;
    decltype(&mbu_stem_fp32) stem;
    decltype(&mbu_classifier_fp32) classifier;
    PyObject *device, *stream;
} g;

using c10::DispatchKey;
using c10::DispatchKeySet;

// no mode, transform or subclass has a say in what torch.empty() returns
bool ordinary()
{
    const DispatchKeySet ignored =
        DispatchKeySet({DispatchKey::BackendSelect, DispatchKey::ADInplaceOrView}) | c10::autocast_dispatch_keyset;
    return (c10::impl::tls_local_dispatch_key_set().included_.raw_repr() & ~ignored.raw_repr()) == 0 &&
           !at::impl::torch_function_mode_enabled();
}

const at::Tensor *plain(PyObject *o, at::ScalarType dtype, int dim)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    const DispatchKeySet known({DispatchKey::CUDA, DispatchKey::ADInplaceOrView, DispatchKey::AutogradCUDA,
                                DispatchKey::AutocastCUDA});
    if (!t.defined() || !t.is_cuda() || (t.key_set().raw_repr() & ~known.raw_repr()) != 0 || t.scalar_type() != dtype || t.dim() < dim ||
        !t.is_contiguous())
        return nullptr;
    return &t;
}

bool whole(PyObject *o, int &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long x = PyLong_AsLongAndOverflow(o, &over);
    if (over || x < 0 || x > 0x7fffffffL) return false;
    v = (int)x;
    return true;
}

bool sizes_fit(const at::Tensor &t)
{
    for (int64_t s : t.sizes())
        if (s > 0x7fffffffLL) return false;
    return true;
}

// the current stream's handle (raises in a forked child, as torch.empty() does)
void *current_stream(const at::Tensor &t)
{
    torch::utils::maybe_initialize_device(t.device());
    PyObject *d = PyObject_CallNoArgs(g.device);
    if (!d) throw python_error();
    PyObject *s = PyObject_CallOneArg(g.stream, d);
    Py_DECREF(d);
    if (!s) throw python_error();
    void *p = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    if (!p && PyErr_Occurred()) throw python_error();
    return p;
}

at::Tensor make(at::IntArrayRef shape, at::ScalarType dtype, c10::Device device)
{
    return at::empty(shape, at::TensorOptions().dtype(dtype).device(device));
}

// What a call takes from an input.  Read while the interpreter lock is held, together with the checks:
// another thread may give the tensor other data (x.data = y, resize_) as soon as the lock is released.
template <typename T> struct Input {
    const T *p;
    int d[4];          // sizes of the first four dimensions
    c10::Device device;
    explicit Input(const at::Tensor &t) : p((const T *)t.data_ptr()), d{}, device(t.device())
    {
        const at::IntArrayRef sizes = t.sizes();
        for (size_t i = 0; i < sizes.size() && i < 4; ++i) d[i] = (int)sizes[i];
    }
};
template <typename T> const T *pointer(const at::Tensor &t) { return (const T *)t.data_ptr(); }
uint32_t *out_words(const at::Tensor &t) { return t.defined() ? (uint32_t *)t.data_ptr() : nullptr; }

// the tuple of the two outputs (None for one that was not asked for), or the error code
PyObject *result(int rc, const at::Tensor &a, const at::Tensor &b)
{
    if (rc != MBU_OK) return PyLong_FromLong(rc);
    PyObject *x = THPVariable_Wrap(a), *y = b.defined() ? THPVariable_Wrap(b) : Py_NewRef(Py_None);
    PyObject *r = x && y ? PyTuple_Pack(2, x, y) : nullptr;
    Py_XDECREF(x);
    Py_XDECREF(y);
    return r;
}
PyObject *result(int rc, const at::Tensor &a) { return rc != MBU_OK ? PyLong_FromLong(rc) : THPVariable_Wrap(a); }

// allocates and calls without the interpreter lock, as a foreign-function call does: `f` reads no input tensor
template <typename F> int unlocked(F &&f)
{
    struct Lock {
        PyThreadState *s = PyEval_SaveThread();
        ~Lock() { PyEval_RestoreThread(s); }
    } lock;
    return f();
}

// (act, cin, packed_w, cout, thresh) -> (bits, None)
PyObject *conv(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int cin, cout;
    if (n != 5 || !g.stream || !ordinary()) Py_RETURN_NONE;
    const at::Tensor *act = plain(a[0], at::kInt, 4), *w = plain(a[2], at::kByte, 0), *th = plain(a[4], at::kInt, 0);
    if (!act || !w || !th || act->dim() != 4 || !sizes_fit(*act) || !whole(a[1], cin) || !whole(a[3], cout)) Py_RETURN_NONE;
    const Input<uint32_t> x(*act);
    const void *const blob = pointer<uint8_t>(*w);
    const int32_t *const theta = pointer<int32_t>(*th);
    void *s = current_stream(*act);
    at::Tensor bits;
    const int rc = unlocked([&] {
        bits = make({x.d[0], x.d[1], x.d[2], cout / 32}, at::kInt, x.device);
        return g.conv(x.p, x.d[0], x.d[1], x.d[2], cin, blob, cout, theta, out_words(bits), nullptr, s);
    });
    return result(rc, bits, at::Tensor());
    END_HANDLE_TH_ERRORS
}

// (act, cin, packed_w, cout, thresh) -> (bits, None)
PyObject *tconv(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int cin, cout;
    if (n != 5 || !g.stream || !ordinary()) Py_RETURN_NONE;
    const at::Tensor *act = plain(a[0], at::kInt, 4), *w = plain(a[2], at::kByte, 0), *th = plain(a[4], at::kInt, 0);
    if (!act || !w || !th || act->dim() != 4 || !sizes_fit(*act) || !whole(a[1], cin) || !whole(a[3], cout)) Py_RETURN_NONE;
    const Input<uint32_t> x(*act);
    const void *const blob = pointer<uint8_t>(*w);
    const int32_t *const theta = pointer<int32_t>(*th);
    void *s = current_stream(*act);
    at::Tensor bits;
    const int rc = unlocked([&] {
        bits = make({x.d[0], 2LL * x.d[1], 2LL * x.d[2], cout / 32}, at::kInt, x.device);
        return g.tconv(x.p, x.d[0], x.d[1], x.d[2], cin, blob, cout, theta, out_words(bits), nullptr, s);
    });
    return result(rc, bits, at::Tensor());
    END_HANDLE_TH_ERRORS
}

// how the second input of a layer enters
enum Second { FUSED, CONCAT, TWO };

// (act, ca, low, clow, upsample, packed_w, cout, thresh, want_pool) -> (bits, pooled bits or None); low may be
// None for FUSED; upsample is read for TWO only
template <Second KIND> PyObject *two_inputs(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int ca, cb, cout;
    if (n != 9 || !g.stream || !ordinary()) Py_RETURN_NONE;
    const at::Tensor *act = plain(a[0], at::kInt, 4), *w = plain(a[5], at::kByte, 0), *th = plain(a[7], at::kInt, 0);
    const bool single = KIND == FUSED && a[2] == Py_None;
    const at::Tensor *low = single ? nullptr : plain(a[2], at::kInt, 4);
    if (!act || !w || !th || (!low && !single) || act->dim() != 4 || !sizes_fit(*act) || (low && !sizes_fit(*low)) ||
        !whole(a[1], ca) || !whole(a[3], cb) || !whole(a[6], cout) || !PyBool_Check(a[4]) || !PyBool_Check(a[8]))
        Py_RETURN_NONE;
    const bool up = a[4] == Py_True, want_pool = a[8] == Py_True;
    const Input<uint32_t> x(*act), y(single ? *act : *low);
    const void *const blob = pointer<uint8_t>(*w);
    const int32_t *const theta = pointer<int32_t>(*th);
    const uint32_t *const pb = single ? nullptr : y.p;
    void *s = current_stream(*act);
    at::Tensor bits, pool;
    const int rc = unlocked([&] {
        const int N = x.d[0], H = x.d[1], W = x.d[2];
        bits = make({N, H, W, cout / 32}, at::kInt, x.device);
        if (want_pool) pool = make({N, H / 2, W / 2, cout / 32}, at::kInt, x.device);
        uint32_t *const ob = out_words(bits), *const op = out_words(pool);
        if (KIND == FUSED) return g.fused(x.p, ca, pb, cb, N, H, W, blob, cout, theta, ob, op, s);
        if (KIND == CONCAT) return g.concat(x.p, ca, pb, cb, N, H, W, blob, cout, theta, ob, op, s);
        return g.two(x.p, ca, pb, cb, y.d[1], y.d[2], up ? 1 : 0, N, H, W, blob, cout, theta, ob, op, s);
    });
    return result(rc, bits, pool);
    END_HANDLE_TH_ERRORS
}

// (x) -> bits
PyObject *pack(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 1 || !g.stream || !ordinary()) Py_RETURN_NONE;
    const at::Tensor *f = plain(a[0], at::kFloat, 4), *t = f ? f : plain(a[0], at::kChar, 4);
    if (!t || t->dim() != 4 || !sizes_fit(*t)) Py_RETURN_NONE;
    const Input<char> x(*t);
    const int dtype = f ? 1 : 0;
    void *s = current_stream(*t);
    at::Tensor bits;
    const int rc = unlocked([&] {
        bits = make({x.d[0], x.d[1], x.d[2], (x.d[3] + 31LL) / 32}, at::kInt, x.device);
        return g.pack(x.p, dtype, x.d[0], x.d[1], x.d[2], x.d[3], out_words(bits), s);
    });
    return result(rc, bits);
    END_HANDLE_TH_ERRORS
}

// (image, w) -> (bits, None)
PyObject *stem(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 2 || !g.stream || !ordinary()) Py_RETURN_NONE;
    const at::Tensor *image = plain(a[0], at::kFloat, 4), *wt = plain(a[1], at::kFloat, 1);
    if (!image || !wt || image->dim() != 4 || !sizes_fit(*image) || !sizes_fit(*wt)) Py_RETURN_NONE;
    const Input<float> x(*image), w(*wt);
    void *s = current_stream(*image);
    at::Tensor bits;
    const int rc = unlocked([&] {
        bits = make({x.d[0], x.d[2], x.d[3], w.d[0] / 32}, at::kInt, x.device);
        return g.stem(x.p, x.d[0], x.d[1], x.d[2], x.d[3], w.p, w.d[0], out_words(bits), nullptr, s);
    });
    return result(rc, bits, at::Tensor());
    END_HANDLE_TH_ERRORS
}

// (act, c, w, b) -> logits
PyObject *classifier(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int c;
    if (n != 4 || !g.stream || !ordinary()) Py_RETURN_NONE;
    const at::Tensor *act = plain(a[0], at::kInt, 4), *wt = plain(a[2], at::kFloat, 1), *bias = plain(a[3], at::kFloat, 0);
    if (!act || !wt || !bias || act->dim() != 4 || !sizes_fit(*act) || !sizes_fit(*wt) || !whole(a[1], c)) Py_RETURN_NONE;
    const Input<uint32_t> x(*act);
    const Input<float> w(*wt);
    const float *const b = pointer<float>(*bias);
    void *s = current_stream(*act);
    at::Tensor out;
    const int rc = unlocked([&] {
        out = make({x.d[0], w.d[0], x.d[1], x.d[2]}, at::kFloat, x.device);
        return g.classifier(x.p, x.d[0], x.d[1], x.d[2], c, w.p, b, w.d[0], (float *)out.data_ptr(), s);
    });
    return result(rc, out);
    END_HANDLE_TH_ERRORS
}

// (addresses of the eight C-ABI functions in the order of `g`, current device, current raw stream of a device)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 10) {
        PyErr_SetString(PyExc_TypeError, "bind: eight addresses and two functions");
        return nullptr;
    }
    void *p[8];
    for (int i = 0; i < 8; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: null address");
            return nullptr;
        }
    }
    g.conv = (decltype(g.conv))p[0];
    g.fused = (decltype(g.fused))p[1];
    g.concat = (decltype(g.concat))p[2];
    g.two = (decltype(g.two))p[3];
    g.tconv = (decltype(g.tconv))p[4];
    g.pack = (decltype(g.pack))p[5];
    g.stem = (decltype(g.stem))p[6];
    g.classifier = (decltype(g.classifier))p[7];
    Py_XSETREF(g.device, Py_NewRef(a[8]));
    Py_XSETREF(g.stream, Py_NewRef(a[9]));
    Py_RETURN_NONE;
}

#define MBU_METHOD(name, f) {name, (PyCFunction)(void (*)(void))(f), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    MBU_METHOD("bind", bind), MBU_METHOD("conv", conv), MBU_METHOD("fused", two_inputs<FUSED>),
    MBU_METHOD("concat", two_inputs<CONCAT>), MBU_METHOD("two_inputs", two_inputs<TWO>), MBU_METHOD("tconv", tconv),
    MBU_METHOD("pack", pack), MBU_METHOD("stem", stem), MBU_METHOD("classifier", classifier),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
