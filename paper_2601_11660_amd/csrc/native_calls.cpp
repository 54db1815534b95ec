// The single-layer calls of binding.py without Python in between: argument checks, the output tensors and
// the C-ABI call.  A call of a small layer is bound by its host side: of 6.5 us the launch takes 3.4, and in
// Python the output tensor took 1.5, marshalling 0.6, the checks 0.5 and the stream 0.2; here all of these take 1.3
// (a 64->64 layer at 64x64 6.6 -> 4.8 us, the other small calls 6.1-7.2 -> 4.8-5.1).
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

at::Tensor make(at::IntArrayRef shape, at::ScalarType dtype, const at::Tensor &like)
{
    return at::empty(shape, at::TensorOptions().dtype(dtype).device(like.device()));
}

const uint32_t *words(const at::Tensor &t) { return (const uint32_t *)t.data_ptr(); }
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

// allocates and calls without the interpreter lock, as a foreign-function call does
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
    void *s = current_stream(*act);
    at::Tensor bits;
    const int rc = unlocked([&] {
        bits = make({act->size(0), act->size(1), act->size(2), cout / 32}, at::kInt, *act);
        return g.conv(words(*act), (int)act->size(0), (int)act->size(1), (int)act->size(2), cin, w->data_ptr(), cout,
                      (const int32_t *)th->data_ptr(), out_words(bits), nullptr, s);
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
    void *s = current_stream(*act);
    at::Tensor bits;
    const int rc = unlocked([&] {
        bits = make({act->size(0), 2 * act->size(1), 2 * act->size(2), cout / 32}, at::kInt, *act);
        return g.tconv(words(*act), (int)act->size(0), (int)act->size(1), (int)act->size(2), cin, w->data_ptr(), cout,
                       (const int32_t *)th->data_ptr(), out_words(bits), nullptr, s);
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
    void *s = current_stream(*act);
    at::Tensor bits, pool;
    const int rc = unlocked([&] {
        const int N = (int)act->size(0), H = (int)act->size(1), W = (int)act->size(2);
        bits = make({N, H, W, cout / 32}, at::kInt, *act);
        if (want_pool) pool = make({N, H / 2, W / 2, cout / 32}, at::kInt, *act);
        const uint32_t *pa = words(*act), *pb = low ? words(*low) : nullptr;
        const int32_t *pt = (const int32_t *)th->data_ptr();
        if (KIND == FUSED) return g.fused(pa, ca, pb, cb, N, H, W, w->data_ptr(), cout, pt, out_words(bits), out_words(pool), s);
        if (KIND == CONCAT) return g.concat(pa, ca, pb, cb, N, H, W, w->data_ptr(), cout, pt, out_words(bits), out_words(pool), s);
        return g.two(pa, ca, pb, cb, (int)low->size(1), (int)low->size(2), up ? 1 : 0, N, H, W, w->data_ptr(), cout, pt,
                     out_words(bits), out_words(pool), s);
    });
    return result(rc, bits, pool);
    END_HANDLE_TH_ERRORS
}

// (x) -> bits
PyObject *pack(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 1 || !g.stream || !ordinary()) Py_RETURN_NONE;
    const at::Tensor *f = plain(a[0], at::kFloat, 4), *x = f ? f : plain(a[0], at::kChar, 4);
    if (!x || x->dim() != 4 || !sizes_fit(*x)) Py_RETURN_NONE;
    void *s = current_stream(*x);
    at::Tensor bits;
    const int rc = unlocked([&] {
        bits = make({x->size(0), x->size(1), x->size(2), (x->size(3) + 31) / 32}, at::kInt, *x);
        return g.pack(x->data_ptr(), f ? 1 : 0, (int)x->size(0), (int)x->size(1), (int)x->size(2), (int)x->size(3),
                      out_words(bits), s);
    });
    return result(rc, bits);
    END_HANDLE_TH_ERRORS
}

// (image, w) -> (bits, None)
PyObject *stem(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 2 || !g.stream || !ordinary()) Py_RETURN_NONE;
    const at::Tensor *x = plain(a[0], at::kFloat, 4), *w = plain(a[1], at::kFloat, 1);
    if (!x || !w || x->dim() != 4 || !sizes_fit(*x) || !sizes_fit(*w)) Py_RETURN_NONE;
    void *s = current_stream(*x);
    at::Tensor bits;
    const int rc = unlocked([&] {
        bits = make({x->size(0), x->size(2), x->size(3), w->size(0) / 32}, at::kInt, *x);
        return g.stem((const float *)x->data_ptr(), (int)x->size(0), (int)x->size(1), (int)x->size(2), (int)x->size(3),
                      (const float *)w->data_ptr(), (int)w->size(0), out_words(bits), nullptr, s);
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
    const at::Tensor *act = plain(a[0], at::kInt, 4), *w = plain(a[2], at::kFloat, 1), *b = plain(a[3], at::kFloat, 0);
    if (!act || !w || !b || act->dim() != 4 || !sizes_fit(*act) || !sizes_fit(*w) || !whole(a[1], c)) Py_RETURN_NONE;
    void *s = current_stream(*act);
    at::Tensor out;
    const int rc = unlocked([&] {
        out = make({act->size(0), w->size(0), act->size(1), act->size(2)}, at::kFloat, *act);
        return g.classifier(words(*act), (int)act->size(0), (int)act->size(1), (int)act->size(2), c,
                            (const float *)w->data_ptr(), (const float *)b->data_ptr(), (int)w->size(0),
                            (float *)out.data_ptr(), s);
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
