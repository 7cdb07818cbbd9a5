// Native call path of pipeline.py: takes torch tensors, allocates the output, fills the descriptors and calls the
// C ABI, all in one C++ function per call.
//
// What bounds it: the small layers of a detector run 5-7 us each, and a layer called through Python objects (ctypes
// structures, tensor attributes, a stream object, an output allocation) cost 11-14 us of host time, so a forward called
// layer by layer waited for the host.  Here the same work is one call; the launch itself is most of what is left.
#include <Python.h>

#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "counts.h"
#include "rtoss.h"

namespace {

PyObject* g_rtoss_error = nullptr;  // binding.RtossError

// ---- errors: the C ABI's status as RtossError(status, message), misuse as Python's own exceptions ----
struct PyError {};  // a Python exception is set
[[noreturn]] void raise(PyObject* type, const char* msg)
{
    PyErr_SetString(type, msg);
    throw PyError{};
}
void require(bool ok, const char* msg)
{
    if (!ok) raise(PyExc_AssertionError, msg);
}
void check(rtoss_status st)
{
    if (st == RTOSS_OK) return;
    PyObject* e = PyObject_CallFunction(g_rtoss_error, "is", (int)st, rtoss_last_error());
    if (e) {
        PyErr_SetObject(g_rtoss_error, e);
        Py_DECREF(e);
    }
    throw PyError{};
}
template <typename F> PyObject* guarded(F&& f)
{
    try {
        return f();
    } catch (const PyError&) {
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}
// the ABI call itself runs without the interpreter lock (a full launch queue makes it wait)
template <typename F> void call(F&& f)
{
    rtoss_status st;
    Py_BEGIN_ALLOW_THREADS
    st = f();
    Py_END_ALLOW_THREADS
    check(st);
}

// ---- arguments ----
const at::Tensor& tensor(PyObject* o)
{
    if (!THPVariable_Check(o)) raise(PyExc_TypeError, "a torch tensor is expected");
    return THPVariable_Unpack(o);
}
long integer(PyObject* o)
{
    const long v = PyLong_AsLong(o);  // (numpy integers and booleans convert through __index__)
    if (v == -1 && PyErr_Occurred()) throw PyError{};
    return v;
}
bool truth(PyObject* o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw PyError{};
    return v != 0;
}
at::ScalarType scalar_type(int dt)
{
    switch (dt) {
    case RTOSS_F32: return at::kFloat;
    case RTOSS_F16: return at::kHalf;
    case RTOSS_BF16: return at::kBFloat16;
    }
    raise(PyExc_KeyError, "unknown dtype");
}
void* current_stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }
void* stream_arg(PyObject* o)
{
    if (o == Py_None) return current_stream();
    void* s = PyLong_AsVoidPtr(o);
    if (!s && PyErr_Occurred()) throw PyError{};
    return s;
}
// The device's own allocation function, at the end of at::empty's dispatch (which costs 0.5 us of a 4 us call).
at::Tensor allocate(at::IntArrayRef shape, at::ScalarType st, const at::Device& dev)
{
    return at::Tensor(at::detail::empty_cuda(shape, st, dev, std::nullopt));
}

// a dictionary: contiguous array of uint16
void acquire_masks(PyObject* o, Py_buffer* view)
{
    if (PyObject_GetBuffer(o, view, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS)) throw PyError{};
    if (view->itemsize != 2 || !view->format || std::strcmp(view->format, "H") != 0) {
        PyBuffer_Release(view);
        raise(PyExc_TypeError, "the dictionary must be an array of uint16");
    }
}
struct Masks {
    Py_buffer view{};
    explicit Masks(PyObject* o) { acquire_masks(o, &view); }
    ~Masks() { PyBuffer_Release(&view); }
    const uint16_t* data() const { return (const uint16_t*)view.buf; }
    int size() const { return (int)(view.len / 2); }
};

// ---- a layer's descriptor and dictionary, where the Python layer object keeps them ----
// (Buffers of its own attributes, not copies: a field of the descriptor or an entry of the dictionary that the program
// changes counts from the next call on, as it does for the calls that go through ctypes.)
struct Layer {
    Py_buffer desc{}, masks{};
    ~Layer()
    {
        PyBuffer_Release(&desc);  // (nothing for a buffer that was not acquired)
        PyBuffer_Release(&masks);
    }
    rtoss_wdesc d() const
    {
        rtoss_wdesc v;
        std::memcpy(&v, desc.buf, sizeof v);
        return v;
    }
    const uint16_t* dict() const { return (const uint16_t*)masks.buf; }
    int P() const { return (int)(masks.len / 2); }
};
constexpr const char* kCapsule = "rtoss.layer";
void free_layer(PyObject* cap) { delete (Layer*)PyCapsule_GetPointer(cap, kCapsule); }
const Layer& layer_of(PyObject* cap)
{
    auto* l = (const Layer*)PyCapsule_GetPointer(cap, kCapsule);
    if (!l) throw PyError{};
    return *l;
}

void arity(Py_ssize_t n, Py_ssize_t want)
{
    if (n != want) raise(PyExc_TypeError, "wrong number of arguments");
}

// layer(wdesc, masks) -> capsule
PyObject* py_layer(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        arity(n, 2);
        auto l = std::make_unique<Layer>();
        if (PyObject_GetBuffer(a[0], &l->desc, PyBUF_SIMPLE)) throw PyError{};
        if (l->desc.len != sizeof(rtoss_wdesc)) raise(PyExc_TypeError, "the descriptor must be a WDesc");
        acquire_masks(a[1], &l->masks);
        PyObject* cap = PyCapsule_New(l.get(), kCapsule, free_layer);
        if (!cap) throw PyError{};
        l.release();
        return cap;
    });
}

struct Spatial {
    int64_t N, H, W, C;
};
Spatial spatial_of(const at::Tensor& x, bool nchw)
{
    if (x.dim() != 4) raise(PyExc_ValueError, "activations have 4 dimensions");
    const auto s = x.sizes();
    return nchw ? Spatial{s[0], s[2], s[3], s[1]} : Spatial{s[0], s[1], s[2], s[3]};
}

at::Tensor new_output(const rtoss_wdesc& d, const Spatial& x, long stride, bool nchw, int out_dt, const at::Device& dev)
{
    const int64_t p = 2 * (d.ksize / 2) - d.ksize;
    const int64_t Ho = (x.H + p) / stride + 1, Wo = (x.W + p) / stride + 1;
    if (nchw) return allocate({x.N, d.Co, Ho, Wo}, scalar_type(out_dt), dev);
    return allocate({x.N, Ho, Wo, d.Co}, scalar_type(out_dt), dev);
}

// conv(layer, blob, x, stride, relu, out_dt, y, layout, coherent)
PyObject* py_conv(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        arity(n, 9);
        const Layer& l = layer_of(a[0]);
        const rtoss_wdesc d = l.d();
        const at::Tensor &blob = tensor(a[1]), &x = tensor(a[2]);
        const long stride = integer(a[3]);
        const bool relu = truth(a[4]), coherent = truth(a[8]);
        const int out_dt = a[5] == Py_None ? (int)d.dt : (int)integer(a[5]);
        const int layout = (int)integer(a[7]);
        require(x.is_cuda() && x.is_contiguous(), "x must be a contiguous cuda tensor");
        const bool nchw = layout == RTOSS_NCHW;
        const Spatial xs = spatial_of(x, nchw);
        require(xs.C == d.Ci, "x has another number of channels than the layer");
        at::Tensor y;
        void* yp = nullptr;
        if (a[6] != Py_None) yp = tensor(a[6]).data_ptr();
        else if (stride > 0) {  // (a bad stride is the library's error to report)
            y = new_output(d, xs, stride, nchw, out_dt, x.device());
            yp = y.data_ptr();
        }
        const rtoss_cdesc c{(int)xs.N, (int)xs.H, (int)xs.W, (int)stride, d.ksize / 2, (rtoss_layout)layout, (rtoss_dtype)out_dt, relu ? 1 : 0};
        void* s = current_stream();
        const void *bp = blob.data_ptr(), *xp = x.data_ptr();
        call([&] {
            return coherent ? rtoss_conv2d_pattern_coherent(&d, &c, nullptr, l.dict(), l.P(), bp, xp, yp, s)
                            : rtoss_conv2d_pattern(&d, &c, l.dict(), l.P(), bp, xp, yp, s);
        });
        if (a[6] != Py_None) {
            Py_INCREF(a[6]);
            return a[6];
        }
        return THPVariable_Wrap(std::move(y));
    });
}

// position pitch of a channels-last tensor or of a channel slice of one (0: plain)
int pitch_of(const at::Tensor& t)
{
    const auto z = t.sizes(), st = t.strides();
    const int64_t ld = st[2];
    require(st[3] == 1 && st[1] == z[2] * ld && st[0] == z[1] * z[2] * ld, "not a channel slice");
    return ld == z[3] ? 0 : (int)ld;
}
const float* per_channel(PyObject* o, int Co)
{
    if (o == Py_None) return nullptr;
    const at::Tensor& t = tensor(o);
    require(t.is_cuda() && t.scalar_type() == at::kFloat && t.numel() == Co, "scale and bias are float32 cuda tensors of Co elements");
    return (const float*)t.data_ptr();
}

// conv_fused(layer, blob, x, stride, scale, bias, act, residual, out_dt, y)
PyObject* py_conv_fused(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        arity(n, 10);
        const Layer& l = layer_of(a[0]);
        const rtoss_wdesc d = l.d();
        const at::Tensor &blob = tensor(a[1]), &x = tensor(a[2]);
        const long stride = integer(a[3]);
        const int out_dt = a[8] == Py_None ? (int)d.dt : (int)integer(a[8]);
        require(x.is_cuda() && x.is_contiguous(), "x must be a contiguous cuda tensor");
        const Spatial xs = spatial_of(x, false);
        require(xs.C == d.Ci, "x has another number of channels than the layer");
        if (stride < 1) raise(stride ? PyExc_ValueError : PyExc_ZeroDivisionError, "stride must be positive");
        rtoss_epilogue e{};
        e.scale_dev = per_channel(a[4], d.Co);
        e.bias_dev = per_channel(a[5], d.Co);
        e.act = (rtoss_act)integer(a[6]);
        at::Tensor made;
        if (a[9] == Py_None) made = new_output(d, xs, stride, false, out_dt, x.device());
        const at::Tensor& y = a[9] == Py_None ? made : tensor(a[9]);
        if (a[9] != Py_None) {
            const int64_t p = 2 * (d.ksize / 2) - d.ksize;
            const auto z = y.sizes();
            require(y.dim() == 4 && z[0] == xs.N && z[1] == (xs.H + p) / stride + 1 && z[2] == (xs.W + p) / stride + 1 &&
                        z[3] == d.Co && y.scalar_type() == scalar_type(out_dt),
                    "y has the wrong shape or dtype");
            e.y_ld = pitch_of(y);
        }
        if (a[7] != Py_None) {
            const at::Tensor& r = tensor(a[7]);
            require(r.is_cuda() && r.sizes() == y.sizes() && r.scalar_type() == y.scalar_type(), "residual must have y's shape and dtype");
            e.residual_dev = r.data_ptr();
            e.residual_ld = pitch_of(r);
        }
        const rtoss_cdesc c{(int)xs.N, (int)xs.H, (int)xs.W, (int)stride, d.ksize / 2, RTOSS_NHWC, (rtoss_dtype)out_dt, 0};
        void* s = current_stream();
        const void *bp = blob.data_ptr(), *xp = x.data_ptr();
        void* yp = y.data_ptr();
        call([&] { return rtoss_conv2d_pattern_fused(&d, &c, &e, l.dict(), l.P(), bp, xp, yp, s); });
        if (a[9] != Py_None) {
            Py_INCREF(a[9]);
            return a[9];
        }
        return THPVariable_Wrap(std::move(made));
    });
}

// an index tensor of exactly G entries: `t` itself, or its first G
PyObject* first_entries(PyObject* o, int64_t G)
{
    const at::Tensor& t = tensor(o);
    if (t.dim() == 1 && t.size(0) == G) {
        Py_INCREF(o);
        return o;
    }
    return THPVariable_Wrap(t.slice(0, 0, G));
}

// select(w, dt, masks) -> idx
PyObject* py_select(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        arity(n, 3);
        const at::Tensor& w = tensor(a[0]);
        const int dt = (int)integer(a[1]);
        Masks m(a[2]);
        require(w.is_cuda() && w.is_contiguous(), "w must be a contiguous cuda tensor");
        const int64_t G = w.numel() / 9;
        at::Tensor idx = allocate({G > 0 ? G : 1}, at::kByte, w.device());
        void* s = current_stream();
        const void* wp = w.data_ptr();
        auto* ip = (uint8_t*)idx.data_ptr();
        call([&] { return rtoss_select_patterns(wp, (rtoss_dtype)dt, w.numel(), m.data(), m.size(), ip, s); });
        if (G == 0) idx = idx.slice(0, 0, 0);
        return THPVariable_Wrap(std::move(idx));
    });
}

// A sequence argument's elements as they are at the start of the call, held until it returns.  (A list can be changed by
// any Python code that runs meanwhile: attribute lookups here, other threads while the ABI call is without the lock.)
struct Seq {
    PyObject* o;
    explicit Seq(PyObject* s) : o(PySequence_Tuple(s))
    {
        if (!o) throw PyError{};
    }
    Seq(const Seq&) = delete;
    ~Seq() { Py_DECREF(o); }
    Py_ssize_t size() const { return PyTuple_GET_SIZE(o); }
    PyObject* operator[](Py_ssize_t i) const { return PyTuple_GET_ITEM(o, i); }
};
struct Owned {
    PyObject* o;
    explicit Owned(PyObject* p) : o(p)
    {
        if (!o) throw PyError{};
    }
    Owned(Owned&& other) noexcept : o(other.release()) {}
    ~Owned() { Py_XDECREF(o); }
    PyObject* release()
    {
        PyObject* p = o;
        o = nullptr;
        return p;
    }
};

// select_batch(ws, dt, masks, idxs or None, stream or None) -> list of index tensors
PyObject* py_select_batch(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        arity(n, 5);
        Seq ws(a[0]);
        const int dt = (int)integer(a[1]);
        Masks m(a[2]);
        const bool given = a[3] != Py_None;
        Owned made(PyList_New(0));
        if (!given)
            for (Py_ssize_t i = 0; i < ws.size(); ++i) {
                const at::Tensor& w = tensor(ws[i]);
                Owned t(THPVariable_Wrap(allocate({std::max<int64_t>(w.numel() / 9, 1)}, at::kByte, w.device())));
                if (PyList_Append(made.o, t.o)) throw PyError{};
            }
        Seq idxs(given ? a[3] : made.o);
        const Py_ssize_t count = std::min(ws.size(), idxs.size());
        std::vector<rtoss_select_item> items((size_t)count);
        for (Py_ssize_t i = 0; i < count; ++i) {
            const at::Tensor &w = tensor(ws[i]), &x = tensor(idxs[i]);
            require(w.is_cuda() && w.is_contiguous() && x.is_cuda() && x.numel() >= w.numel() / 9,
                    "weights are contiguous cuda tensors, index tensors have an entry per group");
            items[i] = rtoss_select_item{w.data_ptr(), w.numel(), (uint8_t*)x.data_ptr()};
        }
        void* s = stream_arg(a[4]);
        static const rtoss_select_item none{};
        call([&] { return rtoss_select_patterns_batch(count ? items.data() : &none, (int)count, (rtoss_dtype)dt, m.data(), m.size(), s); });
        Owned out(PyList_New(count));
        for (Py_ssize_t i = 0; i < count; ++i) {
            PyObject* t = first_entries(idxs[i], items[i].n_elems / 9);
            if (!t) throw PyError{};
            PyList_SET_ITEM(out.o, i, t);
        }
        return out.release();
    });
}

// pack_batch(layers, ws, idxs, stream or None); the layers are objects with _native, _bound and blob (pipeline.py), of one dictionary
PyObject* py_pack_batch(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        arity(n, 4);
        static PyObject* const k_native = PyUnicode_InternFromString("_native");
        static PyObject* const k_bound = PyUnicode_InternFromString("_bound");
        static PyObject* const k_blob = PyUnicode_InternFromString("blob");
        Seq layers(a[0]), ws(a[1]), idxs(a[2]);
        const Py_ssize_t count = std::min(layers.size(), std::min(ws.size(), idxs.size()));
        std::vector<rtoss_pack_item> items((size_t)count);
        std::vector<Owned> held;  // the layers' attributes: replacing one during the call must not free it
        held.reserve(3 * (size_t)count);
        const Layer* first = nullptr;
        for (Py_ssize_t i = 0; i < count; ++i) {
            held.emplace_back(PyObject_GetAttr(layers[i], k_native));
            if (held.back().o == Py_None) held.emplace_back(PyObject_CallMethodNoArgs(layers[i], k_bound));
            const Layer& l = layer_of(held.back().o);
            if (!first) first = &l;
            held.emplace_back(PyObject_GetAttr(layers[i], k_blob));
            const at::Tensor &b = tensor(held.back().o), &w = tensor(ws[i]), &x = tensor(idxs[i]);
            require(w.is_cuda() && w.is_contiguous() && x.is_cuda(), "weights and indices are cuda tensors, weights contiguous");
            items[i] = rtoss_pack_item{l.d(), w.data_ptr(), (const uint8_t*)x.data_ptr(), b.data_ptr(), (size_t)b.nbytes()};
        }
        void* s = stream_arg(a[3]);
        if (first) call([&] { return rtoss_pack_batch(items.data(), (int)count, first->dict(), first->P(), s); });
        Py_RETURN_NONE;
    });
}

// histogram(idx, P, hist or None) -> hist
PyObject* py_histogram(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&]() -> PyObject* {
        arity(n, 3);
        const at::Tensor& idx = tensor(a[0]);
        const int P = (int)integer(a[1]);
        require(idx.is_cuda() && idx.scalar_type() == at::kByte && idx.is_contiguous(), "idx must be a contiguous uint8 cuda tensor");
        at::Tensor made;
        const bool fresh = a[2] == Py_None;
        if (fresh) made = allocate({P}, at::kInt, idx.device());
        const at::Tensor& hist = a[2] == Py_None ? made : tensor(a[2]);
        void* s = current_stream();
        const auto* ip = (const uint8_t*)idx.data_ptr();
        auto* hp = (uint32_t*)hist.data_ptr();
        call([&] {
            // (a P that the library refuses is the library's error to report)
            if (fresh && P >= 1 && P <= 255)
                if (const rtoss_status st = rtoss::clear_counts(hp, P, (hipStream_t)s)) return st;
            return rtoss_pattern_histogram(ip, idx.numel(), P, hp, s);
        });
        if (a[2] != Py_None) {
            Py_INCREF(a[2]);
            return a[2];
        }
        return THPVariable_Wrap(std::move(made));
    });
}

// set_error_type(RtossError)
PyObject* py_set_error_type(PyObject*, PyObject* type)
{
    Py_INCREF(type);
    Py_XSETREF(g_rtoss_error, type);
    Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {FAST(layer), FAST(conv), FAST(conv_fused), FAST(select), FAST(select_batch), FAST(pack_batch), FAST(histogram),
                          {"set_error_type", py_set_error_type, METH_O, nullptr},
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host(void) { return PyModule_Create(&kModule); }
