// Native call path of the Python binding (module `_native`): unpacks torch tensors, checks them, allocates the output
// and enqueues the call of include/ss.h on torch's current stream.
//
// A call of the binding is a handful of microseconds of GPU work for the small layers of a network, so the argument
// handling in front of it decides how fast a loop over layers runs: through ctypes (17 converted arguments, two size
// queries, a stream object) a call took 13.4 us on the host, more than the kernel of every layer below about 10 us;
// through this module it takes 4.1 to 4.8 (3x3 64 -> 64 on one 16x16 image, which takes the GPU 2.8 a call).
//
// Contract with binding.py: a function here either does the whole call and returns its result, or does nothing and
// returns None.  None means "not the plain good case" -- a wrong type, size or device, an option that is not handled
// here, or arguments that the library refuses -- and the caller then takes its own checked path, which finds and reports the
// reason.  A call that may have enqueued its kernel and failed all the same returns (status, row, block): made again, an
// update would move the weights twice, and a residual that is also the output would be added twice.
#include <Python.h>
#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <hip/hip_runtime_api.h>
#include <torch/csrc/autograd/python_variable.h>
#include <list>
#include <mutex>
#include <vector>
#include "../../include/ss.h"

namespace {

// ---------------------------------------------------------------------------------------------
// argument helpers: all return false for anything that is not the plain good case
// ---------------------------------------------------------------------------------------------
bool read_desc(PyObject *o, ss_weight_desc *d)
{
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return false;
    }
    const bool ok = b.len == (Py_ssize_t)sizeof(*d);
    if (ok) memcpy(d, b.buf, sizeof(*d));
    PyBuffer_Release(&b);
    return ok;
}

bool read_int(PyObject *o, int32_t *v)
{
    if (!PyLong_Check(o)) return false;
    const long x = PyLong_AsLong(o);
    if (x == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    if (x < INT32_MIN || x > INT32_MAX) return false;
    *v = (int32_t)x;
    return true;
}

bool read_pair(PyObject *o, int32_t *a, int32_t *b)
{
    return PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == 2 && read_int(PyTuple_GET_ITEM(o, 0), a) &&
           read_int(PyTuple_GET_ITEM(o, 1), b);
}

// A contiguous device tensor; nullptr otherwise.
const at::Tensor *dev_tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.is_cuda() && t.layout() == at::kStrided && t.is_contiguous() ? &t : nullptr;
}

// An optional fp32 vector of at least n values: *p = its address or NULL for None.
bool read_vector(PyObject *o, int64_t n, const float **p)
{
    *p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor *t = dev_tensor(o);
    if (!t || t->scalar_type() != at::kFloat || t->numel() < n) return false;
    *p = static_cast<const float *>(t->const_data_ptr());
    return true;
}

bool type_fits(int32_t dtype, at::ScalarType st)
{
    switch (dtype) {
        case SS_F16: return st == at::kHalf;
        case SS_BF16: return st == at::kBFloat16;
        case SS_I8: return st == at::kChar;
        case SS_F8: return st == at::kByte || st == at::kFloat8_e4m3fn;
        default: return false;
    }
}

bool weight_type_fits(int32_t dtype, at::ScalarType st)
{
    if (dtype == SS_I8 || dtype == SS_F8) return st == at::kChar || st == at::kByte || st == at::kFloat8_e4m3fn;
    return st == at::kHalf || st == at::kBFloat16 || st == at::kShort || st == at::kUInt16;
}

// The output: `o` when given (shape and type checked), a new tensor on x's device otherwise.
bool output(PyObject *o, const at::Tensor &x, at::IntArrayRef shape, at::ScalarType st, at::Tensor *y)
{
    if (o == Py_None) {
        *y = at::detail::empty_cuda(shape, st, x.device(), c10::nullopt);
        return true;
    }
    const at::Tensor *t = dev_tensor(o);
    if (!t || t->scalar_type() != st || t->sizes() != shape) return false;
    *y = *t;
    return true;
}

// The result of a call that is enqueued: from here on nothing may end in None.
PyObject *give(PyObject *o, const at::Tensor &y)
{
    if (o != Py_None) {
        Py_INCREF(o);
        return o;
    }
    try {
        return THPVariable_Wrap(y);
    } catch (const std::exception &e) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// The answer for a status other than SS_OK (bad: row and block of an invalid mask, or NULL): the library checks its arguments before
// it enqueues anything, the other two statuses come afterwards.
PyObject *refuse(int st, const int32_t *bad = nullptr)
{
    if (st != SS_ERR_HIP && st != SS_ERR_BAD_MASK) Py_RETURN_NONE;
    return Py_BuildValue("(iii)", st, bad ? bad[0] : -1, bad ? bad[1] : -1);
}

// A call into the library with the interpreter lock given up, as ctypes does it: a launch blocks while the stream's queue is full,
// and a compression waits.  The operands belong to the caller's arguments or to tensors held here; nothing in the library throws.
template <typename F>
int unlocked(F &&f)
{
    PyThreadState *const ts = PyEval_SaveThread();
    const int st = f();
    PyEval_RestoreThread(ts);
    return st;
}

// ---------------------------------------------------------------------------------------------
// Workspaces of the split reduction for callers that hand none over.  A workspace starts zero and every call hands its
// ticket counters back at zero, so one per stream serves all calls on that stream; calls on different streams never
// share one, and two threads on one stream are ordered by the stream.  At most kMaxPool of them (each at most about
// 16 MiB) are kept, the least recently used one goes first; its memory returns to torch's allocator, which hands it out
// again in the order of the stream it was allocated on.  Under graph capture the caller's own path allocates a
// workspace that belongs to the graph.
// ---------------------------------------------------------------------------------------------
struct PoolEntry {
    int device;
    hipStream_t stream;
    at::Tensor ws;
};
constexpr size_t kMaxPool = 8;
std::mutex pool_mutex;
std::list<PoolEntry> &pool()
{
    static auto *p = new std::list<PoolEntry>;      // never destroyed: its tensors must not outlive torch's allocator
    return *p;
}

bool pooled_workspace(const at::Tensor &x, hipStream_t s, size_t need, at::Tensor *ws)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return false;
    const std::lock_guard<std::mutex> lock(pool_mutex);
    auto &l = pool();
    for (auto it = l.begin(); it != l.end(); ++it)
        if (it->device == x.get_device() && it->stream == s) {
            if ((size_t)it->ws.numel() < need) {
                l.erase(it);
                break;
            }
            l.splice(l.begin(), l, it);
            *ws = it->ws;
            return true;
        }
    if (l.size() >= kMaxPool) l.pop_back();
    l.push_front({(int)x.get_device(), s, at::zeros({(int64_t)need}, x.options().dtype(at::kByte))});
    *ws = l.front().ws;
    return true;
}

// ---------------------------------------------------------------------------------------------
// convolution
// ---------------------------------------------------------------------------------------------
enum ConvKind { kSparse = 0, kDense = 1, kQ8Sparse = 2, kQ8Dense = 3 };

int call_conv(int kind, const ss_weight_desc *d, const void *x, const int32_t *nhw, const void *w, const float *scale,
              const float *bias, const void *residual, const int32_t *sp, int32_t act, void *y, void *ws, size_t ws_bytes,
              void *stream)
{
    switch (kind) {
        case kSparse:
            return ss_conv2d_res_fwd(d, x, nhw[0], nhw[1], nhw[2], w, bias, residual, sp[0], sp[1], sp[2], sp[3], act, y, ws,
                                     ws_bytes, stream);
        case kDense:
            return ss_conv2d_dense_res_fwd(d, x, nhw[0], nhw[1], nhw[2], w, bias, residual, sp[0], sp[1], sp[2], sp[3], act, y,
                                           ws, ws_bytes, stream);
        case kQ8Sparse:
            return ss_conv2d_q8_fwd(d, x, nhw[0], nhw[1], nhw[2], w, scale, bias, sp[0], sp[1], sp[2], sp[3], act, SS_F16, y,
                                    ws, ws_bytes, stream);
        default:
            return ss_conv2d_q8_dense_fwd(d, x, nhw[0], nhw[1], nhw[2], w, scale, bias, sp[0], sp[1], sp[2], sp[3], act, SS_F16,
                                          y, ws, ws_bytes, stream);
    }
}

bool read_image(const ss_weight_desc &d, const at::Tensor *x, int32_t *nhw)
{
    if (!x || x->dim() != 4 || !type_fits(d.dtype, x->scalar_type()) || x->size(3) != d.cin) return false;
    for (int i = 0; i < 3; i++) {
        if (x->size(i) <= 0 || x->size(i) > INT32_MAX) return false;
        nhw[i] = (int32_t)x->size(i);
    }
    return true;
}

bool out_size(const ss_weight_desc &d, const int32_t *nhw, const int32_t *sp, int64_t *ho, int64_t *wo)
{
    if (sp[0] <= 0 || sp[1] <= 0 || sp[2] < 0 || sp[3] < 0) return false;
    const int64_t h = (int64_t)nhw[1] + 2 * (int64_t)sp[2] - d.kh, w = (int64_t)nhw[2] + 2 * (int64_t)sp[3] - d.kw;
    if (h < 0 || w < 0) return false;
    *ho = h / sp[0] + 1;
    *wo = w / sp[1] + 1;
    return true;
}

bool weights_fit(const ss_weight_desc &d, bool sparse, const at::Tensor *w)
{
    size_t need = 0;
    return w && (sparse ? ss_packed_bytes(&d, &need) : ss_dense_bytes(&d, &need)) == SS_OK && w->nbytes() >= need;
}

// conv(kind, desc, x, weights, scale, bias, residual, stride, pad, act, y, workspace) -> y, (status, row, block) or None
PyObject *conv(PyObject *const *a, Py_ssize_t n)
{
    int32_t kind, act, sp[4], nhw[3];
    ss_weight_desc d;
    if (n != 12 || !read_int(a[0], &kind) || !read_desc(a[1], &d) || !read_pair(a[7], &sp[0], &sp[1]) ||
        !read_pair(a[8], &sp[2], &sp[3]) || !read_int(a[9], &act))
        Py_RETURN_NONE;
    const bool sparse = kind == kSparse || kind == kQ8Sparse, q8 = kind == kQ8Sparse || kind == kQ8Dense;
    const at::Tensor *x = dev_tensor(a[2]), *w = dev_tensor(a[3]);
    int64_t ho, wo;
    const float *scale, *bias;
    if (!read_image(d, x, nhw) || !out_size(d, nhw, sp, &ho, &wo) || !weights_fit(d, sparse, w) ||
        !read_vector(a[4], d.cout, &scale) || !read_vector(a[5], d.cout, &bias))
        Py_RETURN_NONE;
    const int64_t shape[4] = {nhw[0], ho, wo, d.cout};
    const at::ScalarType yt = q8 ? at::kHalf : x->scalar_type();
    const void *residual = nullptr;
    if (a[6] != Py_None) {
        const at::Tensor *r = dev_tensor(a[6]);
        if (!r || r->scalar_type() != yt || r->sizes() != at::IntArrayRef(shape, 4)) Py_RETURN_NONE;
        residual = r->const_data_ptr();
    }
    at::Tensor y, ws;
    if (!output(a[10], *x, at::IntArrayRef(shape, 4), yt, &y)) Py_RETURN_NONE;
    const hipStream_t s = c10::hip::getCurrentHIPStream().stream();
    size_t ws_bytes = 0;
    void *wsp = nullptr;
    if (a[11] != Py_None) {
        const at::Tensor *t = dev_tensor(a[11]);
        if (!t) Py_RETURN_NONE;
        wsp = t->data_ptr();
        ws_bytes = t->nbytes();
    }
    const void *xp = x->const_data_ptr(), *wp = w->const_data_ptr();
    void *yp = y.data_ptr();
    const auto call = [&] { return call_conv(kind, &d, xp, nhw, wp, scale, bias, residual, sp, act, yp, wsp, ws_bytes, s); };
    int st = unlocked(call);
    if (st == SS_ERR_WORKSPACE && a[11] == Py_None) {     // (nothing is enqueued yet; few calls need one)
        size_t need = 0;
        if (ss_conv2d_workspace_bytes(&d, nhw[0], nhw[1], nhw[2], sp[0], sp[1], sp[2], sp[3], &need) != SS_OK ||
            !pooled_workspace(*x, s, need, &ws))
            Py_RETURN_NONE;
        wsp = ws.data_ptr();
        ws_bytes = ws.nbytes();
        st = unlocked(call);
    }
    return st == SS_OK ? give(a[10], y) : refuse(st);
}

// fused(sparse, desc1, x, w1, bias1, stride, pad, act1, desc2, w2, bias2, residual, act2, y) -> y, (status, row, block) or None
PyObject *fused(PyObject *const *a, Py_ssize_t n)
{
    int32_t sparse, act1, act2, sp[4], nhw[3];
    ss_weight_desc d1, d2;
    if (n != 14 || !read_int(a[0], &sparse) || !read_desc(a[1], &d1) || !read_pair(a[5], &sp[0], &sp[1]) ||
        !read_pair(a[6], &sp[2], &sp[3]) || !read_int(a[7], &act1) || !read_desc(a[8], &d2) || !read_int(a[12], &act2))
        Py_RETURN_NONE;
    const at::Tensor *x = dev_tensor(a[2]), *w1 = dev_tensor(a[3]), *w2 = dev_tensor(a[9]);
    int64_t ho, wo;
    const float *b1, *b2;
    if (!read_image(d1, x, nhw) || !out_size(d1, nhw, sp, &ho, &wo) || !weights_fit(d1, sparse != 0, w1) ||
        !weights_fit(d2, sparse != 0, w2) || !read_vector(a[4], d1.cout, &b1) || !read_vector(a[10], d2.cout, &b2))
        Py_RETURN_NONE;
    const int64_t shape[4] = {nhw[0], ho, wo, d2.cout};
    const void *residual = nullptr;
    if (a[11] != Py_None) {
        const at::Tensor *r = dev_tensor(a[11]);
        if (!r || r->scalar_type() != x->scalar_type() || r->sizes() != at::IntArrayRef(shape, 4)) Py_RETURN_NONE;
        residual = r->const_data_ptr();
    }
    at::Tensor y;
    if (!output(a[13], *x, at::IntArrayRef(shape, 4), x->scalar_type(), &y)) Py_RETURN_NONE;
    const auto fn = sparse ? ss_conv2d_pw_fused_fwd : ss_conv2d_pw_fused_dense_fwd;
    const void *xp = x->const_data_ptr(), *w1p = w1->const_data_ptr(), *w2p = w2->const_data_ptr();
    void *yp = y.data_ptr();
    const hipStream_t s = c10::hip::getCurrentHIPStream().stream();
    const int st = unlocked([&] {
        return fn(&d1, xp, nhw[0], nhw[1], nhw[2], w1p, b1, sp[0], sp[1], sp[2], sp[3], act1, &d2, w2p, b2, residual, act2, yp, s);
    });
    return st == SS_OK ? give(a[13], y) : refuse(st);
}

// ---------------------------------------------------------------------------------------------
// pooling and depthwise convolution
// ---------------------------------------------------------------------------------------------
// maxpool(x, k, stride, pad, y) -> y, (status, row, block) or None
PyObject *maxpool(PyObject *const *a, Py_ssize_t n)
{
    int32_t k, s, pad;
    if (n != 5 || !read_int(a[1], &k) || !read_int(a[2], &s) || !read_int(a[3], &pad)) Py_RETURN_NONE;
    const at::Tensor *x = dev_tensor(a[0]);
    if (!x || x->dim() != 4 || (x->scalar_type() != at::kHalf && x->scalar_type() != at::kBFloat16) || s <= 0 || pad < 0)
        Py_RETURN_NONE;
    const int64_t h = x->size(1) + 2 * (int64_t)pad - k, w = x->size(2) + 2 * (int64_t)pad - k;
    if (h < 0 || w < 0 || x->numel() == 0 || x->size(0) > INT32_MAX || x->size(1) > INT32_MAX || x->size(2) > INT32_MAX || x->size(3) > INT32_MAX)
        Py_RETURN_NONE;
    at::Tensor y;
    if (!output(a[4], *x, {x->size(0), h / s + 1, w / s + 1, x->size(3)}, x->scalar_type(), &y)) Py_RETURN_NONE;
    const int32_t d[4] = {(int32_t)x->size(0), (int32_t)x->size(1), (int32_t)x->size(2), (int32_t)x->size(3)};
    const int32_t dtype = x->scalar_type() == at::kHalf ? SS_F16 : SS_BF16;
    const void *xp = x->const_data_ptr();
    void *yp = y.data_ptr();
    const hipStream_t stream = c10::hip::getCurrentHIPStream().stream();
    const int st = unlocked([&] { return ss_maxpool2d(xp, d[0], d[1], d[2], d[3], dtype, k, s, pad, yp, stream); });
    return st == SS_OK ? give(a[4], y) : refuse(st);
}

// dwconv(x, w, bias, pad, act, y) -> y, (status, row, block) or None
PyObject *dwconv(PyObject *const *a, Py_ssize_t n)
{
    int32_t ph, pw, act;
    if (n != 6 || !read_pair(a[3], &ph, &pw) || !read_int(a[4], &act)) Py_RETURN_NONE;
    const at::Tensor *x = dev_tensor(a[0]), *w = dev_tensor(a[1]);
    if (!x || !w || x->dim() != 4 || w->dim() != 3 || (x->scalar_type() != at::kHalf && x->scalar_type() != at::kBFloat16) ||
        w->scalar_type() != x->scalar_type() || w->size(2) != x->size(3) || x->numel() == 0 || x->size(0) > INT32_MAX ||
        x->size(1) > INT32_MAX || x->size(2) > INT32_MAX || x->size(3) > INT32_MAX || w->size(0) > 4096 || w->size(1) > 4096)
        Py_RETURN_NONE;
    const float *bias;
    if (!read_vector(a[2], x->size(3), &bias)) Py_RETURN_NONE;
    const int64_t ho = x->size(1) + 2 * (int64_t)ph - w->size(0) + 1, wo = x->size(2) + 2 * (int64_t)pw - w->size(1) + 1;
    if (ho <= 0 || wo <= 0) Py_RETURN_NONE;
    at::Tensor y;
    if (!output(a[5], *x, {x->size(0), ho, wo, x->size(3)}, x->scalar_type(), &y)) Py_RETURN_NONE;
    const int32_t d[4] = {(int32_t)x->size(0), (int32_t)x->size(1), (int32_t)x->size(2), (int32_t)x->size(3)};
    const int32_t dtype = x->scalar_type() == at::kHalf ? SS_F16 : SS_BF16, kh = (int32_t)w->size(0), kw = (int32_t)w->size(1);
    const void *xp = x->const_data_ptr(), *wp = w->const_data_ptr();
    void *yp = y.data_ptr();
    const hipStream_t s = c10::hip::getCurrentHIPStream().stream();
    const int st = unlocked([&] { return ss_dwconv2d_fwd(xp, d[0], d[1], d[2], d[3], dtype, wp, bias, kh, kw, ph, pw, act, yp, s); });
    return st == SS_OK ? give(a[5], y) : refuse(st);
}

// ---------------------------------------------------------------------------------------------
// packing
// ---------------------------------------------------------------------------------------------
// pack(mode, desc, W, U, M, out) -> out, (status, row, block) or None; mode 0: compress, 1: update and compress,
// 2: dense (M may be None)
PyObject *pack(PyObject *const *a, Py_ssize_t n)
{
    int32_t mode;
    ss_weight_desc d;
    if (n != 6 || !read_int(a[0], &mode) || !read_desc(a[1], &d) || d.cout <= 0 || d.cin <= 0 || d.kh <= 0 || d.kw <= 0) Py_RETURN_NONE;
    const __int128 count = (__int128)d.cout * d.cin * d.kh * d.kw;
    const at::Tensor *W = dev_tensor(a[2]), *M = a[4] == Py_None ? nullptr : dev_tensor(a[4]), *U = nullptr;
    if (!W || !weight_type_fits(d.dtype, W->scalar_type()) || W->numel() != count) Py_RETURN_NONE;
    if (a[4] == Py_None ? mode != 2 : (!M || (M->scalar_type() != at::kByte && M->scalar_type() != at::kBool) || M->numel() != count))
        Py_RETURN_NONE;
    if (mode == 1) {
        U = dev_tensor(a[3]);
        if (!U || U->scalar_type() != W->scalar_type() || U->numel() != count || d.dtype == SS_I8 || d.dtype == SS_F8) Py_RETURN_NONE;
    }
    size_t need = 0;
    if ((mode == 2 ? ss_dense_bytes(&d, &need) : ss_packed_bytes(&d, &need)) != SS_OK) Py_RETURN_NONE;
    at::Tensor out;
    if (a[5] == Py_None) {
        out = at::detail::empty_cuda({(int64_t)need}, at::kByte, W->device(), c10::nullopt);
    } else {
        const at::Tensor *t = dev_tensor(a[5]);
        if (!t || t->nbytes() < need) Py_RETURN_NONE;
        out = *t;
    }
    const hipStream_t s = c10::hip::getCurrentHIPStream().stream();
    const uint8_t *m = M ? static_cast<const uint8_t *>(M->const_data_ptr()) : nullptr;
    // (an update writes W: an address for writing, so that a lazy clone parts from what it shares memory with)
    void *wp = mode == 1 ? W->mutable_data_ptr() : const_cast<void *>(W->const_data_ptr());
    const void *up = U ? U->const_data_ptr() : nullptr;
    void *op = out.data_ptr();
    int32_t bad[2] = {-1, -1};
    const int st = unlocked([&] {               // (the compressing calls wait for the stream)
        if (mode == 2) return ss_dense_pack(&d, wp, m, op, s);
        if (mode == 1) return ss_mask_update_compress(&d, wp, up, m, op, bad, s);
        return ss_mask_compress(&d, wp, m, op, bad, s);
    });
    return st == SS_OK ? give(a[5], out) : refuse(st, bad);
}

// ---------------------------------------------------------------------------------------------
// Prepared launches: the arguments of a call, marshalled once by the binding; calling the object enqueues it on torch's
// current stream.
// ---------------------------------------------------------------------------------------------
struct Launch {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    PyObject *keep;            // everything the addresses below belong to
    PyObject *on_error;        // called with the status of a call that failed
    int kind;                  // ConvKind, or 4 / 5: fused pair (sparse / dense), 6: max pooling, 7 / 8: fused pair and a third layer, 9: convolution and its pooling (at ws)
    ss_weight_desc d1, d2, d3;
    const void *w3;
    const float *b3;
    void *y3;
    int32_t act3;
    const void *x, *w1, *w2, *residual;
    const float *scale, *b1, *b2;
    void *y, *ws;
    size_t ws_bytes;
    int32_t nhw[3], sp[4], act1, act2;
    int32_t pool[3];           // channels, dtype, k (stride and padding in sp)
};

PyObject *launch_call(PyObject *self, PyObject *const *, size_t, PyObject *)
{
    Launch *l = reinterpret_cast<Launch *>(self);
    hipStream_t s;
    try {
        s = c10::hip::getCurrentHIPStream().stream();
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    const int st = unlocked([&] {
        if (l->kind <= kQ8Dense)
            return call_conv(l->kind, &l->d1, l->x, l->nhw, l->w1, l->scale, l->b1, l->residual, l->sp, l->act1, l->y, l->ws, l->ws_bytes, s);
        if (l->kind == 6)
            return ss_maxpool2d(l->x, l->nhw[0], l->nhw[1], l->nhw[2], l->pool[0], l->pool[1], l->pool[2], l->sp[0], l->sp[2], l->y, s);
        if (l->kind == 9)
            return ss_conv2d_maxpool_dense_fwd(&l->d1, l->x, l->nhw[0], l->nhw[1], l->nhw[2], l->w1, l->b1, l->sp[0], l->sp[1], l->sp[2], l->sp[3], l->act1,
                                               l->y, l->ws, s);
        if (l->kind >= 7) {
            const auto fn = l->kind == 7 ? ss_conv2d_pw2_fused_fwd : ss_conv2d_pw2_fused_dense_fwd;
            return fn(&l->d1, l->x, l->nhw[0], l->nhw[1], l->nhw[2], l->w1, l->b1, l->sp[0], l->sp[1], l->sp[2], l->sp[3], l->act1, &l->d2,
                      l->w2, l->b2, l->residual, l->act2, l->y, &l->d3, l->w3, l->b3, l->act3, l->y3, s);
        }
        const auto fn = l->kind == 4 ? ss_conv2d_pw_fused_fwd : ss_conv2d_pw_fused_dense_fwd;
        return fn(&l->d1, l->x, l->nhw[0], l->nhw[1], l->nhw[2], l->w1, l->b1, l->sp[0], l->sp[1], l->sp[2], l->sp[3], l->act1, &l->d2,
                  l->w2, l->b2, l->residual, l->act2, l->y, s);
    });
    if (st != SS_OK) return PyObject_CallFunction(l->on_error, "i", st);
    Py_RETURN_NONE;
}

int launch_traverse(PyObject *self, visitproc visit, void *arg)
{
    Launch *l = reinterpret_cast<Launch *>(self);
    Py_VISIT(l->keep);
    Py_VISIT(l->on_error);
    return 0;
}

int launch_clear(PyObject *self)
{
    Launch *l = reinterpret_cast<Launch *>(self);
    Py_CLEAR(l->keep);
    Py_CLEAR(l->on_error);
    return 0;
}

void launch_dealloc(PyObject *self)
{
    PyObject_GC_UnTrack(self);
    launch_clear(self);
    Py_TYPE(self)->tp_free(self);
}

PyTypeObject LaunchType = {PyVarObject_HEAD_INIT(nullptr, 0)};

bool address(PyObject *o, void **p)      // an int, or None for NULL
{
    *p = nullptr;
    if (o == Py_None) return true;
    *p = PyLong_AsVoidPtr(o);
    return !PyErr_Occurred();
}

// launch(kind, desc1, desc2 | None, (x, w1, w2, scale, b1, b2, residual, y, ws) addresses, ws_bytes,
//        (N, H, W), (sh, sw, ph, pw), act1, act2, (C, dtype, k) | None, (desc3, w3, b3, act3, y3) | None, keep, on_error) -> callable
PyObject *launch(PyObject *, PyObject *args)
{
    int kind, act1, act2, nhw[3], sp[4], pool3[3] = {0, 0, 0};
    PyObject *d1, *d2, *ptrs, *poolo, *third, *keep, *on_error;
    Py_ssize_t ws_bytes;
    if (!PyArg_ParseTuple(args, "iOOO!n(iii)(iiii)iiOOOO", &kind, &d1, &d2, &PyTuple_Type, &ptrs, &ws_bytes, &nhw[0], &nhw[1], &nhw[2],
                          &sp[0], &sp[1], &sp[2], &sp[3], &act1, &act2, &poolo, &third, &keep, &on_error))
        return nullptr;
    if (kind < 0 || kind > 9 || (kind == 7 || kind == 8) != (third != Py_None) || PyTuple_GET_SIZE(ptrs) != 9) {
        PyErr_SetString(PyExc_ValueError, "launch: bad kind or address list");
        return nullptr;
    }
    if (poolo != Py_None && !PyArg_ParseTuple(poolo, "iii", &pool3[0], &pool3[1], &pool3[2])) return nullptr;
    ss_weight_desc w1{}, w2{};
    if ((d1 != Py_None && !read_desc(d1, &w1)) || (d2 != Py_None && !read_desc(d2, &w2))) {
        PyErr_SetString(PyExc_ValueError, "launch: bad descriptor");
        return nullptr;
    }
    void *p[9];
    for (int i = 0; i < 9; i++)
        if (!address(PyTuple_GET_ITEM(ptrs, i), &p[i])) return nullptr;
    ss_weight_desc last{};
    void *w3 = nullptr, *b3 = nullptr, *y3 = nullptr;
    int act3 = 0;
    if (third != Py_None) {
        PyObject *d3, *pw, *pb, *py;
        if (!PyArg_ParseTuple(third, "OOOiO", &d3, &pw, &pb, &act3, &py) || !address(pw, &w3) || !address(pb, &b3) || !address(py, &y3)) return nullptr;
        if (!read_desc(d3, &last)) {
            PyErr_SetString(PyExc_ValueError, "launch: bad descriptor");
            return nullptr;
        }
    }
    PyObject *o = LaunchType.tp_alloc(&LaunchType, 0);
    if (!o) return nullptr;
    Launch *l = reinterpret_cast<Launch *>(o);
    l->vectorcall = reinterpret_cast<vectorcallfunc>(launch_call);
    Py_INCREF(keep);
    Py_INCREF(on_error);
    l->keep = keep;
    l->on_error = on_error;
    l->kind = kind;
    l->d1 = w1;
    l->d2 = w2;
    l->d3 = last;
    l->w3 = w3;
    l->b3 = static_cast<const float *>(b3);
    l->y3 = y3;
    l->act3 = act3;
    l->x = p[0]; l->w1 = p[1]; l->w2 = p[2];
    l->scale = static_cast<const float *>(p[3]);
    l->b1 = static_cast<const float *>(p[4]);
    l->b2 = static_cast<const float *>(p[5]);
    l->residual = p[6]; l->y = p[7]; l->ws = p[8];
    l->ws_bytes = (size_t)ws_bytes;
    for (int i = 0; i < 3; i++) { l->nhw[i] = nhw[i]; l->pool[i] = pool3[i]; }
    for (int i = 0; i < 4; i++) l->sp[i] = sp[i];
    l->act1 = act1;
    l->act2 = act2;
    return o;
}

// Every entry point runs inside this: what torch throws (a tensor without storage under torch.func, symbolic sizes, no memory)
// must not leave through the interpreter's C frames, where it would end the process.  The caller's path meets it again and reports it.
// (Not `catch (...)`: a daemon thread that asks for the interpreter lock while the interpreter shuts down is ended by a forced
// unwind, which has to pass.)
template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyObject *entry(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    try {
        return F(a, n);
    } catch (const std::exception &) {
    }
    PyErr_Clear();                              // (torch's Python errors leave theirs set)
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"conv", reinterpret_cast<PyCFunction>(entry<conv>), METH_FASTCALL, nullptr},
    {"fused", reinterpret_cast<PyCFunction>(entry<fused>), METH_FASTCALL, nullptr},
    {"maxpool", reinterpret_cast<PyCFunction>(entry<maxpool>), METH_FASTCALL, nullptr},
    {"dwconv", reinterpret_cast<PyCFunction>(entry<dwconv>), METH_FASTCALL, nullptr},
    {"pack", reinterpret_cast<PyCFunction>(entry<pack>), METH_FASTCALL, nullptr},
    {"launch", launch, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Native call path of the binding.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    LaunchType.tp_name = "paper_2411_00288_amd._native.Launch";
    LaunchType.tp_basicsize = sizeof(Launch);
    LaunchType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL;
    LaunchType.tp_vectorcall_offset = offsetof(Launch, vectorcall);
    LaunchType.tp_call = PyVectorcall_Call;
    LaunchType.tp_traverse = launch_traverse;
    LaunchType.tp_clear = launch_clear;
    LaunchType.tp_dealloc = launch_dealloc;
    if (PyType_Ready(&LaunchType) < 0) return nullptr;
    return PyModule_Create(&module);
}
