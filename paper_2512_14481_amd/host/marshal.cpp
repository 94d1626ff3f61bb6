// Argument marshalling of the Python binding in native code (module _marshal): the checks of binding.py, device pointers and sizes
// out of torch tensors, the current HIP stream, and the call of the C entry point.
//
// A call through ctypes costs 5 to 8 us of the host's time beside the launches, as much as a small call's kernels run: one
// scale-training step of a 64 x 256 -> 256 linear, six kernels of 21 us in five calls, took 47 us.
//
// Every function returns the entry point's status, or None for arguments that it does not take as they are: another type than a plain
// tensor, int, float, tuple or list, a tensor that is not on the device or not contiguous, a failed check.  The caller then runs the
// checks in Python, which name the fault.  Nothing is kept from one call to the next but the entry points' addresses.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>

#include "sasq.h"

namespace {

struct Entry {
    decltype(&sasq_fakequant_fwd) fakequant_fwd;
    decltype(&sasq_fakequant_bwd) fakequant_bwd;
    decltype(&sasq_fakequant_fwd_batch) fakequant_fwd_batch;
    decltype(&sasq_fakequant_bwd_batch) fakequant_bwd_batch;
    decltype(&sasq_fakequant_fwd_pc_batch) fakequant_fwd_pc_batch;
    decltype(&sasq_fakequant_bwd_pc_batch) fakequant_bwd_pc_batch;
    decltype(&sasq_scale_sgd) scale_sgd;
    decltype(&sasq_scale_sgd_vec) scale_sgd_vec;
    decltype(&sasq_scale_adamw) scale_adamw;
    decltype(&sasq_static_linear) static_linear;
    decltype(&sasq_static_linear_batch) static_linear_batch;
    decltype(&sasq_static_linear_grouped) static_linear_grouped;
    decltype(&sasq_packed_weight_bytes) packed_weight_bytes;
    decltype(&sasq_bwd_weight_bytes) bwd_weight_bytes;
    decltype(&sasq_linear_bwd_input) linear_bwd_input;
    decltype(&sasq_absmax_scale) absmax_scale;
    decltype(&sasq_quantize_weight) quantize_weight;
    decltype(&sasq_pack_weight) pack_weight;
    decltype(&sasq_prepare_bwd_weight) prepare_bwd_weight;
};
Entry entry{};

struct NotTaken {};                                        // leave the call to the Python checks

void want(bool ok)
{
    if (!ok) throw NotTaken{};
}

const at::Tensor& tensor(PyObject* o)
{
    want(THPVariable_CheckExact(o));
    const at::Tensor& t = THPVariable_Unpack(o);
    want(t.is_cuda() && t.is_contiguous());
    return t;
}

const at::Tensor* optional_tensor(PyObject* o) { return o == Py_None ? nullptr : &tensor(o); }

const at::Tensor& tensor(PyObject* o, at::ScalarType type)
{
    const at::Tensor& t = tensor(o);
    want(t.scalar_type() == type);
    return t;
}

template <typename T = void>
T* pointer(const at::Tensor& t) { return static_cast<T*>(t.data_ptr()); }

template <typename T = void>
T* pointer(const at::Tensor* t) { return t ? pointer<T>(*t) : nullptr; }

template <typename T>
T* pointer(PyObject* o, at::ScalarType type) { return o == Py_None ? nullptr : pointer<T>(tensor(o, type)); }

float* floats(PyObject* o) { return pointer<float>(tensor(o, at::kFloat)); }

int64_t integer(PyObject* o)
{
    want(PyLong_CheckExact(o));
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    want(overflow == 0);
    return v;
}

int small(PyObject* o)
{
    const int64_t v = integer(o);
    want(v == static_cast<int>(v));
    return static_cast<int>(v);
}

double real(PyObject* o)
{
    want(PyFloat_CheckExact(o));
    return PyFloat_AS_DOUBLE(o);
}

sasq_dtype dtype_of(const at::Tensor& x)
{
    want(x.scalar_type() == at::kHalf || x.scalar_type() == at::kBFloat16);
    return x.scalar_type() == at::kHalf ? SASQ_F16 : SASQ_BF16;
}

void same(const at::Tensor& a, const at::Tensor& x) { want(a.scalar_type() == x.scalar_type() && a.sizes() == x.sizes()); }

int64_t row_length(const at::Tensor& x)
{
    want(x.dim() >= 1);
    return x.numel() / (x.size(0) > 1 ? x.size(0) : 1);
}

size_t bytes(const at::Tensor& t) { return static_cast<size_t>(t.numel()) * t.element_size(); }
size_t bytes(const at::Tensor* t) { return t ? bytes(*t) : 0; }

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Runs an entry point without the interpreter's lock, as a call through ctypes does: a launch may wait for room in its queue.
template <typename Call>
int unlocked(Call&& call)
{
    void* st = current_stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call(st);
    Py_END_ALLOW_THREADS
    return rc;
}

bool blocked(int wf) { return wf == SASQ_W_INT8_BLOCKED || wf == SASQ_W_INT4_BLOCKED; }

// [M, K] activations, [M, N] outputs and a weight of N rows in format wf
struct Linear {
    int64_t M, N, K;
    sasq_dtype dt;
};
Linear linear_shape(const at::Tensor& x, const at::Tensor& wq, const at::Tensor& s_w, const at::Tensor* bias, const at::Tensor& y, int wf)
{
    want(x.dim() == 2 && y.dim() == 2);
    Linear l{x.size(0), y.size(1), x.size(1), dtype_of(x)};
    want(wq.scalar_type() == at::kChar || wq.scalar_type() == at::kByte);
    if (blocked(wf)) want(static_cast<size_t>(wq.numel()) == entry.packed_weight_bytes(l.N, l.K, static_cast<sasq_wfmt>(wf)));
    else             want(wq.dim() == 2 && wq.size(0) == l.N && wq.size(1) == (wf == SASQ_W_INT8 ? l.K : l.K / 2));
    want(y.size(0) == l.M && y.scalar_type() == x.scalar_type() && s_w.numel() == l.N && (!bias || bias->numel() == l.N));
    return l;
}

int fakequant_fwd(PyObject* const* a)                      // x, s, y, codes, bits
{
    const at::Tensor &x = tensor(a[0]), &y = tensor(a[2]);
    float* s = floats(a[1]);
    auto* codes = pointer<int8_t>(a[3], at::kChar);
    same(y, x);
    const int bits = small(a[4]);
    const sasq_dtype dt = dtype_of(x);
    const int64_t cols = row_length(x), rows = x.size(0);
    void *xp = pointer(x), *yp = pointer(y);
    return unlocked([&](void* st) { return entry.fakequant_fwd(xp, s, yp, codes, rows, cols, bits, dt, st); });
}

int fakequant_bwd(PyObject* const* a)                      // x, dy, s, dx, ds, workspace, bits
{
    const at::Tensor &x = tensor(a[0]), &dy = tensor(a[1]), &ws = tensor(a[5]);
    const at::Tensor* dx = optional_tensor(a[3]);
    float *s = floats(a[2]), *ds = floats(a[4]);
    same(dy, x);
    if (dx) same(*dx, x);
    const int bits = small(a[6]);
    const sasq_dtype dt = dtype_of(x);
    const int64_t cols = row_length(x), rows = x.size(0);
    void *xp = pointer(x), *gp = pointer(dy), *dp = pointer(dx), *wp = pointer(ws);
    const size_t wb = bytes(ws);
    return unlocked([&](void* st) { return entry.fakequant_bwd(xp, gp, s, dp, ds, rows, cols, bits, dt, wp, wb, st); });
}

struct FqItems {
    sasq_fq_item item[SASQ_MAX_BATCH];
    int count;
    sasq_dtype dt;
};
// per_channel: s and ds hold one factor per column
FqItems fq_items(PyObject* list, bool backward, bool per_channel)
{
    want(PyList_CheckExact(list) || PyTuple_CheckExact(list));
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(list);
    want(n >= 1 && n <= SASQ_MAX_BATCH);
    FqItems f{};
    f.count = static_cast<int>(n);
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject* t = PySequence_Fast_GET_ITEM(list, i);
        want(PyTuple_CheckExact(t) && PyTuple_GET_SIZE(t) == (backward ? 5 : 3));
        const at::Tensor &x = tensor(PyTuple_GET_ITEM(t, 0)), &s = tensor(PyTuple_GET_ITEM(t, backward ? 2 : 1), at::kFloat);
        const sasq_dtype dt = dtype_of(x);
        want(i == 0 || dt == f.dt);
        f.dt = dt;
        sasq_fq_item& it = f.item[i];
        it.cols = row_length(x);
        it.rows = x.size(0);
        if (per_channel) want(x.dim() >= 2 && s.numel() == x.size(1));
        if (backward) {
            const at::Tensor &dy = tensor(PyTuple_GET_ITEM(t, 1)), &ds = tensor(PyTuple_GET_ITEM(t, 4), at::kFloat);
            const at::Tensor* dx = optional_tensor(PyTuple_GET_ITEM(t, 3));
            same(dy, x);
            if (dx) same(*dx, x);
            if (per_channel) want(ds.numel() == x.size(1));
            it.dy = pointer(dy);
            it.out = pointer(dx);
            it.ds = pointer<float>(ds);
        } else {
            const at::Tensor& y = tensor(PyTuple_GET_ITEM(t, 2));
            same(y, x);
            it.out = pointer(y);
        }
        it.x = pointer(x);
        it.s = pointer<float>(s);
    }
    return f;
}

template <bool PC>
int fq_fwd_batch(PyObject* const* a)                       // items, bits
{
    const FqItems f = fq_items(a[0], false, PC);
    const int bits = small(a[1]);
    auto* call = PC ? entry.fakequant_fwd_pc_batch : entry.fakequant_fwd_batch;
    return unlocked([&](void* st) { return call(f.item, f.count, bits, f.dt, st); });
}

template <bool PC>
int fq_bwd_batch(PyObject* const* a)                       // items, workspace, bits
{
    const FqItems f = fq_items(a[0], true, PC);
    const at::Tensor& ws = tensor(a[1]);
    const int bits = small(a[2]);
    void* wp = pointer(ws);
    const size_t wb = bytes(ws);
    auto* call = PC ? entry.fakequant_bwd_pc_batch : entry.fakequant_bwd_batch;
    return unlocked([&](void* st) { return call(f.item, f.count, bits, f.dt, wp, wb, st); });
}

int scale_sgd(PyObject* const* a)                          // s, ds, lr
{
    float *s = floats(a[0]), *ds = floats(a[1]);
    const float lr = static_cast<float>(real(a[2]));
    return unlocked([&](void* st) { return entry.scale_sgd(s, ds, lr, st); });
}

int scale_sgd_vec(PyObject* const* a)                      // s, ds, lr
{
    const at::Tensor &s = tensor(a[0], at::kFloat), &ds = tensor(a[1], at::kFloat);
    want(s.numel() == ds.numel());
    const int64_t n = s.numel();
    const float lr = static_cast<float>(real(a[2]));
    auto *sp = pointer<float>(s), *dp = pointer<float>(ds);
    return unlocked([&](void* st) { return entry.scale_sgd_vec(sp, dp, n, lr, st); });
}

int scale_adamw(PyObject* const* a)                        // s, ds, m, v, step, lr, beta1, beta2, eps, weight_decay
{
    float* p[4];
    const int64_t n = tensor(a[0]).numel();
    for (int i = 0; i < 4; ++i) {
        want(tensor(a[i]).numel() == n);
        p[i] = floats(a[i]);
    }
    const int64_t step = integer(a[4]);
    double h[5];
    for (int i = 0; i < 5; ++i) h[i] = real(a[5 + i]);
    return unlocked([&](void* st) { return entry.scale_adamw(p[0], p[1], p[2], p[3], n, step, h[0], h[1], h[2], h[3], h[4], st); });
}

int static_linear(PyObject* const* a)                      // x, s, wq, s_w, bias, y, wf, workspace, acc_out, xq_out, a_bits
{
    const at::Tensor &x = tensor(a[0]), &wq = tensor(a[2]), &s_w = tensor(a[3], at::kFloat), &y = tensor(a[5]);
    const at::Tensor *bias = optional_tensor(a[4]), *ws = optional_tensor(a[7]);
    want(!bias || bias->scalar_type() == at::kFloat);
    float* s = floats(a[1]);
    const int wf = small(a[6]), a_bits = small(a[10]);
    auto* acc = pointer<int32_t>(a[8], at::kInt);
    auto* xq = pointer<int8_t>(a[9], at::kChar);
    const Linear l = linear_shape(x, wq, s_w, bias, y, wf);
    void *xp = pointer(x), *wp = pointer(wq), *yp = pointer(y), *wsp = pointer(ws);
    auto *sw = pointer<float>(s_w), *bp = pointer<float>(bias);
    const size_t wb = bytes(ws);
    return unlocked([&](void* st) {
        return entry.static_linear(xp, s, wp, sw, bp, yp, acc, xq, l.M, l.N, l.K, a_bits, static_cast<sasq_wfmt>(wf), l.dt, wsp, wb, st);
    });
}

int static_linear_grouped(PyObject* const* a)              // x, s_g, wq, s_w, bias, y, group, wf, workspace, f_out, xq_out, a_bits
{
    const at::Tensor &x = tensor(a[0]), &s_g = tensor(a[1], at::kFloat), &wq = tensor(a[2]), &s_w = tensor(a[3], at::kFloat), &y = tensor(a[5]);
    const at::Tensor *bias = optional_tensor(a[4]), *ws = optional_tensor(a[8]);
    want(!bias || bias->scalar_type() == at::kFloat);
    const int64_t group = integer(a[6]);
    const int wf = small(a[7]), a_bits = small(a[11]);
    auto* f = pointer<float>(a[9], at::kFloat);
    auto* xq = pointer<int8_t>(a[10], at::kChar);
    const Linear l = linear_shape(x, wq, s_w, bias, y, wf);
    want(group > 0 && l.K % group == 0 && s_g.numel() == l.K / group);
    void *xp = pointer(x), *wp = pointer(wq), *yp = pointer(y), *wsp = pointer(ws);
    auto *sg = pointer<float>(s_g), *sw = pointer<float>(s_w), *bp = pointer<float>(bias);
    const size_t wb = bytes(ws);
    return unlocked([&](void* st) {
        return entry.static_linear_grouped(xp, sg, wp, sw, bp, yp, f, xq, l.M, l.N, l.K, group, a_bits, static_cast<sasq_wfmt>(wf), l.dt, wsp, wb, st);
    });
}

int static_linear_batch(PyObject* const* a)                // items, wf, workspace, a_bits
{
    PyObject* list = a[0];
    want(PyList_CheckExact(list) || PyTuple_CheckExact(list));
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(list);
    want(n >= 1 && n <= SASQ_MAX_BATCH);
    const int wf = small(a[1]), a_bits = small(a[3]);
    const at::Tensor& ws = tensor(a[2]);
    sasq_linear_item item[SASQ_MAX_BATCH];
    sasq_dtype dt{};
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject* t = PySequence_Fast_GET_ITEM(list, i);
        want(PyTuple_CheckExact(t) && PyTuple_GET_SIZE(t) == 6);
        auto at_ = [&](int k) { return PyTuple_GET_ITEM(t, k); };
        const at::Tensor &x = tensor(at_(0)), &wq = tensor(at_(2)), &s_w = tensor(at_(3), at::kFloat), &y = tensor(at_(5));
        const at::Tensor* bias = optional_tensor(at_(4));
        want(!bias || bias->scalar_type() == at::kFloat);
        const Linear l = linear_shape(x, wq, s_w, bias, y, wf);
        want(i == 0 || l.dt == dt);
        dt = l.dt;
        item[i] = sasq_linear_item{pointer(x), floats(at_(1)), pointer(wq), pointer<float>(s_w), pointer<float>(bias), pointer(y), l.M, l.N, l.K};
    }
    void* wp = pointer(ws);
    const size_t wb = bytes(ws);
    return unlocked([&](void* st) {
        return entry.static_linear_batch(item, static_cast<int>(n), a_bits, static_cast<sasq_wfmt>(wf), dt, wp, wb, st);
    });
}

int linear_bwd_input(PyObject* const* a)                   // dy, wt, dx, K, acc_out
{
    const at::Tensor &dy = tensor(a[0]), &wt = tensor(a[1]), &dx = tensor(a[2]);
    const at::Tensor* acc = optional_tensor(a[4]);
    want(dy.dim() == 2 && dx.dim() == 2);
    const int64_t M = dy.size(0), N = dy.size(1), K = integer(a[3]);
    want(dx.scalar_type() == dy.scalar_type() && dx.size(0) == M && dx.size(1) == K && bytes(wt) == entry.bwd_weight_bytes(N, K));
    want(!acc || (acc->scalar_type() == at::kFloat && acc->dim() == 2 && acc->size(0) == M && acc->size(1) == K));
    const sasq_dtype dt = dtype_of(dy);
    void *gp = pointer(dy), *wp = pointer(wt), *dp = pointer(dx);
    auto* ap = pointer<float>(acc);
    return unlocked([&](void* st) { return entry.linear_bwd_input(gp, wp, dp, ap, M, N, K, dt, st); });
}

int absmax_scale(PyObject* const* a)                       // x, s, workspace, bits
{
    const at::Tensor &x = tensor(a[0]), &ws = tensor(a[2]);
    float* s = floats(a[1]);
    const int bits = small(a[3]);
    const sasq_dtype dt = dtype_of(x);
    const int64_t cols = row_length(x), rows = x.size(0);
    void *xp = pointer(x), *wp = pointer(ws);
    const size_t wb = bytes(ws);
    return unlocked([&](void* st) { return entry.absmax_scale(xp, s, rows, cols, bits, dt, wp, wb, st); });
}

int quantize_weight(PyObject* const* a)                    // w, wq, s_w, wf
{
    const at::Tensor &w = tensor(a[0], at::kFloat), &wq = tensor(a[1]);
    float* s_w = floats(a[2]);
    const auto wf = static_cast<sasq_wfmt>(small(a[3]));
    want(w.dim() == 2);
    const int64_t N = w.size(0), K = w.size(1);
    auto* wp = pointer<float>(w);
    void* qp = pointer(wq);
    return unlocked([&](void* st) { return entry.quantize_weight(wp, qp, s_w, N, K, wf, st); });
}

int pack_weight(PyObject* const* a)                        // wq, packed, N, K, wf_src
{
    const at::Tensor &wq = tensor(a[0]), &packed = tensor(a[1]);
    const int64_t N = integer(a[2]), K = integer(a[3]);
    const int wf = small(a[4]);
    const bool int8 = wf == SASQ_W_INT8;
    want(N > 0 && K > 0 && wq.numel() == N * (int8 ? K : K / 2) &&
         bytes(packed) == entry.packed_weight_bytes(N, K, int8 ? SASQ_W_INT8_BLOCKED : SASQ_W_INT4_BLOCKED));
    void *qp = pointer(wq), *pp = pointer(packed);
    return unlocked([&](void* st) { return entry.pack_weight(qp, pp, N, K, static_cast<sasq_wfmt>(wf), st); });
}

int prepare_bwd_weight(PyObject* const* a)                 // wq, s_w, wt, N, K, wf, sasq_dtype
{
    const at::Tensor &wq = tensor(a[0]), &s_w = tensor(a[1], at::kFloat), &wt = tensor(a[2]);
    const int64_t N = integer(a[3]), K = integer(a[4]);
    const int wf = small(a[5]), dt = small(a[6]);
    want(N > 0 && K > 0 && bytes(wq) == static_cast<size_t>(N) * (wf == SASQ_W_INT8 ? K : K / 2) && s_w.numel() == N &&
         bytes(wt) == entry.bwd_weight_bytes(N, K));
    void *qp = pointer(wq), *tp = pointer(wt);
    auto* sp = pointer<float>(s_w);
    return unlocked([&](void* st) {
        return entry.prepare_bwd_weight(qp, sp, tp, N, K, static_cast<sasq_wfmt>(wf), static_cast<sasq_dtype>(dt), st);
    });
}

template <int (*CALL)(PyObject* const*), int NARGS>
PyObject* method(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    if (nargs != NARGS || !entry.fakequant_fwd) Py_RETURN_NONE;
    try {
        return PyLong_FromLong(CALL(args));
    } catch (const NotTaken&) {
    } catch (const std::exception&) {                      // a tensor without memory of its own: the Python path says so
    }
    Py_RETURN_NONE;
}

// bind({"sasq_...": address, ...}): the entry points of the library that the binding has loaded
PyObject* bind(PyObject*, PyObject* table)
{
    Entry e{};
    auto set = [&](const char* name, auto& slot) {
        PyObject* v = PyDict_Check(table) ? PyDict_GetItemString(table, name) : nullptr;
        void* p = v ? PyLong_AsVoidPtr(v) : nullptr;
        if (!p && !PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "no address for %s", name);
        slot = reinterpret_cast<std::decay_t<decltype(slot)>>(p);
        return p != nullptr;
    };
    const bool ok = set("sasq_fakequant_fwd", e.fakequant_fwd) && set("sasq_fakequant_bwd", e.fakequant_bwd) &&
        set("sasq_fakequant_fwd_batch", e.fakequant_fwd_batch) && set("sasq_fakequant_bwd_batch", e.fakequant_bwd_batch) &&
        set("sasq_fakequant_fwd_pc_batch", e.fakequant_fwd_pc_batch) && set("sasq_fakequant_bwd_pc_batch", e.fakequant_bwd_pc_batch) &&
        set("sasq_scale_sgd", e.scale_sgd) && set("sasq_scale_sgd_vec", e.scale_sgd_vec) && set("sasq_scale_adamw", e.scale_adamw) &&
        set("sasq_static_linear", e.static_linear) && set("sasq_static_linear_batch", e.static_linear_batch) &&
        set("sasq_static_linear_grouped", e.static_linear_grouped) && set("sasq_packed_weight_bytes", e.packed_weight_bytes) &&
        set("sasq_bwd_weight_bytes", e.bwd_weight_bytes) && set("sasq_linear_bwd_input", e.linear_bwd_input) &&
        set("sasq_absmax_scale", e.absmax_scale) && set("sasq_quantize_weight", e.quantize_weight) &&
        set("sasq_pack_weight", e.pack_weight) && set("sasq_prepare_bwd_weight", e.prepare_bwd_weight);
    if (!ok) return nullptr;
    entry = e;
    Py_RETURN_NONE;
}

#define SASQ_METHOD(NAME, CALL, NARGS) \
    {NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&method<CALL, NARGS>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", bind, METH_O, nullptr},
    SASQ_METHOD("sasq_fakequant_fwd", fakequant_fwd, 5),
    SASQ_METHOD("sasq_fakequant_bwd", fakequant_bwd, 7),
    SASQ_METHOD("sasq_fakequant_fwd_batch", fq_fwd_batch<false>, 2),
    SASQ_METHOD("sasq_fakequant_bwd_batch", fq_bwd_batch<false>, 3),
    SASQ_METHOD("sasq_fakequant_fwd_pc_batch", fq_fwd_batch<true>, 2),
    SASQ_METHOD("sasq_fakequant_bwd_pc_batch", fq_bwd_batch<true>, 3),
    SASQ_METHOD("sasq_scale_sgd", scale_sgd, 3),
    SASQ_METHOD("sasq_scale_sgd_vec", scale_sgd_vec, 3),
    SASQ_METHOD("sasq_scale_adamw", scale_adamw, 10),
    SASQ_METHOD("sasq_static_linear", static_linear, 11),
    SASQ_METHOD("sasq_static_linear_batch", static_linear_batch, 4),
    SASQ_METHOD("sasq_static_linear_grouped", static_linear_grouped, 12),
    SASQ_METHOD("sasq_linear_bwd_input", linear_bwd_input, 5),
    SASQ_METHOD("sasq_absmax_scale", absmax_scale, 4),
    SASQ_METHOD("sasq_quantize_weight", quantize_weight, 4),
    SASQ_METHOD("sasq_pack_weight", pack_weight, 5),
    SASQ_METHOD("sasq_prepare_bwd_weight", prepare_bwd_weight, 7),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// ABI: what the module was compiled against, which the binding compares with what it runs on.
PyMODINIT_FUNC PyInit__marshal()
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "ABI", SASQ_MARSHAL_ABI) < 0) Py_CLEAR(m);
    return m;
}
