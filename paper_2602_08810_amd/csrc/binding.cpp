// The native half of the Python binding (host code only, no kernels): the calls that a program makes most often, in their
// usual form, without the interpreter between the tensors and the C entry points.
//
// What bounds it: small calls are bound by the host, since their kernels take 3 to 6 us.  Marshalled in Python, the
// forward call of 16 rows of 256 steps took 15.7 us and a generated token of 64 x 1536 channels 11.2, here 6.6 and 5.0 (its
// kernel's time); training steps, forward and backward: 16 rows of 256 steps 58.6 and 27.4, packed 76 and 35, complex 54 and 35; the
// chained scans and their adjoints 28 and 18.  What is left is the allocation of the outputs and the launches.
//
// A call is taken only where every argument has the usual form: plain strided GPU tensors on the current device with the
// expected types and shapes, contiguous where the general path looks no further, no caller-supplied scratch,
// no mode of the framework that rewrites calls or allocations.  For everything else, wrong arguments among it, the result
// is None and nothing has been done: api.py's general path then takes the call, or refuses it with its own message.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/TensorSubclassLikeUtils.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include <algorithm>
#include <cstring>

#include "../../include/lrnnx.h"

namespace {

// entry points of the library that api.py has loaded (bind: in this order), and what raises its error
struct {
    decltype(&lrnnx_selective_scan_fwd) fwd;
    decltype(&lrnnx_selective_scan_bwd) bwd;
    decltype(&lrnnx_selective_scan_bwd_workspace_bytes) bwd_bytes;
    decltype(&lrnnx_selective_scan_fwd_complex) cfwd;
    decltype(&lrnnx_selective_scan_bwd_complex) cbwd;
    decltype(&lrnnx_selective_step) step;
    decltype(&lrnnx_selective_step_complex) cstep;
    decltype(&lrnnx_lti_diag_scan) lti;
    decltype(&lrnnx_lti_diag_scan_bwd) lti_bwd;
    decltype(&lrnnx_diag_scan) diag;
    decltype(&lrnnx_diag_scan_bwd) diag_bwd;
    decltype(&lrnnx_workspace_bytes) bytes;
} lib = {};
constexpr int kEntries = sizeof(lib) / sizeof(void *);
int64_t ckpt_interval = 0;
PyObject *check_status = nullptr;

// Names of an entry point's parameters, in the order of the Python function (interned when the module is created).
constexpr int kMaxArgs = 20;
struct Names {
    int count;
    const char *text[kMaxArgs];
    PyObject *key[kMaxArgs];
};
enum { F_U, F_DELTA, F_A, F_BM, F_CM, F_D, F_BIAS, F_Z, F_X0, F_DISC, F_SOFTPLUS, F_PATH, F_LAST, F_CKPT, F_OUT, F_CKPT_OUT, F_WS, F_CU };
Names kFwd = {18, {"u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0", "disc", "delta_softplus", "path",
                   "return_last_state", "return_ckpt", "out", "ckpt_out", "workspace", "cu_seqlens"}, {}};
Names kFwdComplex = {18, {"u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "x0", "disc", "delta_softplus",
                          "return_last_state", "out", "return_ckpt", "ckpt_out", "cu_seqlens", "path", "workspace"}, {}};
constexpr int kFwdComplexAt[7] = {16, 11, 13, 12, 14, 17, 15};       // of the arguments from F_PATH on
enum { B_U, B_DELTA, B_A, B_BM, B_CM, B_DY, B_D, B_BIAS, B_Z, B_X0, B_CKPT, B_DISC, B_SOFTPLUS, B_DX0, B_OUTS, B_WS, B_CU, B_PATH, B_LONGEST };
Names kBwd = {19, {"u", "delta", "A", "Bm", "Cm", "dy", "Dskip", "delta_bias", "z", "x0", "ckpt", "disc", "delta_softplus",
                   "want_dx0", "outs", "workspace", "cu_seqlens", "path", "max_seqlen"}, {}};
Names kStep = {12, {"x", "u", "delta", "A", "Bm", "Cm", "Dskip", "delta_bias", "z", "disc", "delta_softplus", "out"}, {}};
Names kLti = {8, {"lam", "v", "x0", "return_last_state", "out", "workspace", "path", "chain_status"}, {}};
Names kLtiBwd = {8, {"lam", "x", "gx", "x0", "want_dx0", "out", "workspace", "chain_status"}, {}};
Names kDiag = {7, {"a", "b", "x0", "return_last_state", "out", "workspace", "chain_status"}, {}};
Names kDiagBwd = {7, {"a", "x", "gx", "x0", "want_dx0", "workspace", "chain_status"}, {}};

// The arguments by position of their names (null: not given).  False for anything that the list of names does not
// cover: unknown, doubled or surplus arguments.
bool gather(const Names &names, PyObject *args, PyObject *kwargs, PyObject **slot) {
    const Py_ssize_t given = PyTuple_GET_SIZE(args);
    if (given > names.count) return false;
    Py_ssize_t by_name = PyDict_GET_SIZE(kwargs);
    for (int i = 0; i < names.count; ++i) {
        slot[i] = i < given ? PyTuple_GET_ITEM(args, i) : nullptr;
        if (i >= given && by_name > 0) {
            slot[i] = PyDict_GetItemWithError(kwargs, names.key[i]);
            if (slot[i]) --by_name;
            else if (PyErr_Occurred()) { PyErr_Clear(); return false; }
        }
    }
    return by_name == 0;
}

bool absent(PyObject *o) { return !o || o == Py_None; }

// a truth value given as one, or its default
bool flag(PyObject *o, bool otherwise, bool &value) {
    value = o ? o == Py_True : otherwise;
    return !o || o == Py_True || o == Py_False;
}

// a mode given by name (or not at all: the first of them)
bool mode(PyObject *o, std::initializer_list<const char *> names, int32_t &code) {
    code = 0;
    if (!o) return true;
    if (!PyUnicode_CheckExact(o)) return false;
    for (const char *n : names) {
        if (PyUnicode_CompareWithASCIIString(o, n) == 0) return true;
        ++code;
    }
    return false;
}
bool disc_mode(PyObject *o, int32_t &code) { return mode(o, {"zoh_s6", "zoh", "bilinear", "dirac"}, code); }
bool path_mode(PyObject *o, int32_t &code) { return mode(o, {"auto", "single_pass", "chunk_carry"}, code); }

// a number of steps, 0 if it is not given
bool steps(PyObject *o, int64_t &value) {
    value = 0;
    if (absent(o)) return true;
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    value = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}

using Shape = c10::SmallVector<int64_t, 5>;

// The tensors of one call.
struct Call {
    c10::DeviceIndex dev = -1;                           // the current device, asked for when a tensor is on any
    // nothing stands between the call and the tensors' memory: no mode that takes over functions or allocations, no tracing
    bool good = !at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set() &&
                !torch::jit::tracer::isTracing();

    // a plain tensor on the current device, or null: not given
    const at::Tensor *tensor(PyObject *o) {
        if (absent(o)) return nullptr;
        if (!THPVariable_CheckExact(o)) { good = false; return nullptr; }
        const at::Tensor &t = THPVariable_Unpack(o);
        if (t.defined() && t.is_cuda() && dev < 0) dev = c10::hip::current_device();
        if (!t.defined() || !t.is_cuda() || t.get_device() != dev || t.layout() != c10::kStrided || at::isTensorSubclassLike(t) ||
            t.is_conj() || t.is_neg() || t._is_zerotensor()) { good = false; return nullptr; }
        return &t;
    }
    const at::Tensor *needed(PyObject *o) {
        const at::Tensor *t = tensor(o);
        if (!t) good = false;
        return t;
    }
    // its memory, if it is contiguous and of this type and shape
    template <class Ptr> void data(const at::Tensor *t, c10::ScalarType type, c10::IntArrayRef shape, Ptr &p) {
        p = nullptr;
        if (!t || !good) return;
        if (t->scalar_type() != type || t->sizes() != shape || !t->is_contiguous()) { good = false; return; }
        p = static_cast<Ptr>(t->data_ptr());
    }
    // rows [B,D,L], or [D,L] of a packed batch
    template <class Ptr> void rows(const at::Tensor *t, c10::ScalarType type, c10::IntArrayRef shape, Ptr &p, int64_t &sb, int64_t &sd) {
        data(t, type, shape, p);
        if (!p) return;
        sd = t->stride(-2);
        sb = t->dim() == 3 ? t->stride(0) : t->size(0) * sd;
    }
    // [B,D] with any strides
    template <class Ptr> void row(const at::Tensor *t, c10::ScalarType type, c10::IntArrayRef shape, Ptr &p, int64_t &sb, int64_t &sd) {
        p = nullptr;
        if (!t || !good) return;
        if (t->scalar_type() != type || t->sizes() != shape) { good = false; return; }
        p = t->data_ptr(); sb = t->stride(0); sd = t->stride(1);
    }
    at::Tensor make(c10::IntArrayRef shape, c10::ScalarType type) const {
        return at::empty(shape, at::TensorOptions().dtype(type).device(c10::Device(c10::kCUDA, dev)));
    }
    // scratch of the call (given back, like every tensor, when the last reference goes)
    template <class Args> at::Tensor scratch(Args &a, size_t bytes) const {
        at::Tensor ws = make({static_cast<int64_t>(bytes)}, at::kByte);
        a.workspace = ws.data_ptr(); a.workspace_bytes = bytes;
        return ws;
    }
    void *stream() const { return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(dev).stream(); }
};

bool fits32(int64_t v) { return v >= 0 && v <= INT32_MAX; }

// The library's verdict on a call: false with the Python error set, if it was refused.
template <class F, class Args> bool launched(F f, const Args &a) {
    PyThreadState *s = PyEval_SaveThread();              // a full queue may keep the launch waiting
    const int status = f(&a);
    PyEval_RestoreThread(s);
    if (status == LRNNX_OK) return true;
    PyObject *r = PyObject_CallFunction(check_status, "i", status);
    Py_XDECREF(r);
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "lrnnx: call refused");
    return false;
}

PyObject *wrap(at::Tensor &t) { return THPVariable_Wrap(std::move(t)); }
PyObject *given(PyObject *o) { Py_INCREF(o); return o; }

// What the selective scans have in common: sizes, the arguments of both passes and the shapes that follow from them.
struct Scan {
    int64_t B = 0, D = 0, L = 0, N = 0, G = 0;
    bool packed = false;
    c10::ScalarType io, state, map_type;
    Shape rows, one_map, maps, bdn, dn, d1, ckpt;        // one_map: of dBm and dCm; maps: of Bm and Cm

    template <bool CPLX, class Args>
    void read(Call &c, Args &a, PyObject *cu_seqlens, const at::Tensor *u, const at::Tensor *delta, const at::Tensor *A, const at::Tensor *Bm,
              const at::Tensor *Cm, const at::Tensor *Dskip, const at::Tensor *bias, const at::Tensor *z, const at::Tensor *x0) {
        const at::Tensor *cu = c.tensor(cu_seqlens);
        packed = cu != nullptr;
        if (!c.good || u->dim() != (packed ? 2 : 3) || A->dim() != 2) { c.good = false; return; }
        if (packed) {
            c.good = cu->scalar_type() == at::kLong && cu->dim() == 1 && cu->is_contiguous() && cu->numel() >= 2;
            if (!c.good) return;
            a.cu_seqlens = static_cast<const int64_t *>(cu->data_ptr());
        }
        B = packed ? cu->numel() - 1 : u->size(0);
        D = u->size(-2); L = u->size(-1); N = A->size(1);
        io = u->scalar_type();
        a.io_dtype = io == at::kBFloat16 ? LRNNX_BF16 : LRNNX_F32;
        state = CPLX ? at::kComplexFloat : at::kFloat;
        // complex maps: complex64 beside float32, pairs on an axis of their own beside bfloat16
        const bool pairs = CPLX && io == at::kBFloat16;
        map_type = CPLX && !pairs ? at::kComplexFloat : io;
        const int lead = packed ? 0 : 1;
        G = 1;
        if (Bm->dim() == lead + 3 + pairs) G = Bm->size(lead);
        if ((io != at::kBFloat16 && io != at::kFloat) || G < 1 || D % G || !fits32(B) || !fits32(D) || !fits32(N)) { c.good = false; return; }
        if (!packed) { rows.push_back(B); one_map.push_back(B); ckpt.push_back(B); }
        rows.append({D, L});
        if (Bm->dim() == lead + 3 + pairs) one_map.push_back(G);
        one_map.append({L, N});
        maps = one_map;
        if (pairs) maps.push_back(2);
        bdn = {B, D, N}; dn = {D, N}; d1 = {D};
        ckpt.append({D, packed ? L / ckpt_interval + B : (L + ckpt_interval - 1) / ckpt_interval, N});
        a.struct_size = sizeof(a);
        a.B = (int32_t)B; a.D = (int32_t)D; a.N = (int32_t)N; a.bc_groups = (int32_t)G; a.L = L;
        c.rows(u, io, rows, a.u, a.u_stride_b, a.u_stride_d);
        c.rows(delta, io, rows, a.delta, a.delta_stride_b, a.delta_stride_d);
        c.rows(z, io, rows, a.z, a.z_stride_b, a.z_stride_d);
        c.data(A, state, dn, a.A);
        c.data(Bm, map_type, maps, a.Bm);
        c.data(Cm, map_type, maps, a.Cm);
        c.data(Dskip, at::kFloat, d1, a.Dskip);
        c.data(bias, at::kFloat, d1, a.delta_bias);
        c.data(x0, state, bdn, a.x0);
    }
};

template <bool CPLX> PyObject *forward(PyObject *args, PyObject *kwargs) {
    PyObject *o[kMaxArgs];
    std::conditional_t<CPLX, lrnnx_ss_fwd_complex_args, lrnnx_ss_fwd_args> a = {};
    Call c;
    bool softplus, want_last, want_ckpt;
    if (!c.good || !gather(CPLX ? kFwdComplex : kFwd, args, kwargs, o)) Py_RETURN_NONE;
    if constexpr (CPLX) {
        PyObject *tail[7];
        for (int i = 0; i < 7; ++i) tail[i] = o[kFwdComplexAt[i]];
        for (int i = 0; i < 7; ++i) o[F_PATH + i] = tail[i];
    }
    if (!disc_mode(o[F_DISC], a.disc) || !path_mode(o[F_PATH], a.path) || !flag(o[F_SOFTPLUS], true, softplus) ||
        !flag(o[F_LAST], false, want_last) || !flag(o[F_CKPT], false, want_ckpt) || !absent(o[F_CKPT_OUT]) || !absent(o[F_WS])) Py_RETURN_NONE;
    a.delta_softplus = softplus;
    const at::Tensor *u = c.needed(o[F_U]), *delta = c.needed(o[F_DELTA]), *A = c.needed(o[F_A]), *Bm = c.needed(o[F_BM]), *Cm = c.needed(o[F_CM]);
    const at::Tensor *Dskip = c.tensor(o[F_D]), *bias = c.tensor(o[F_BIAS]), *z = c.tensor(o[F_Z]), *x0 = c.tensor(o[F_X0]);
    const at::Tensor *out = c.tensor(o[F_OUT]);
    Scan s;
    s.read<CPLX>(c, a, o[F_CU], u, delta, A, Bm, Cm, Dskip, bias, z, x0);
    if (c.good && out) c.rows(out, s.io, s.rows, a.y, a.y_stride_b, a.y_stride_d);
    // (the general path returns views of a packed batch's output, and without anything beside it of another shape with complex A)
    if (!c.good || (s.packed && (out || (CPLX && !want_last && !want_ckpt)))) Py_RETURN_NONE;
    at::Tensor y, last, ckpt, ws;
    if (!out) {
        y = c.make(s.rows, s.io);
        c.rows(&y, s.io, s.rows, a.y, a.y_stride_b, a.y_stride_d);
    }
    if (want_last) { last = c.make(s.bdn, s.state); c.data(&last, s.state, s.bdn, a.x_last); }
    if (want_ckpt) { ckpt = c.make(s.ckpt, s.state); c.data(&ckpt, s.state, s.ckpt, a.ckpt); }
    if (const size_t n = lib.bytes(CPLX ? LRNNX_WS_FWD_COMPLEX : LRNNX_WS_FWD, s.B, s.D, s.N, s.L, a.io_dtype, (int)s.G, s.packed)) ws = c.scratch(a, n);
    a.stream = c.stream();
    bool done;
    if constexpr (CPLX) done = launched(lib.cfwd, a); else done = launched(lib.fwd, a);
    if (!done) return nullptr;
    PyObject *py = out ? given(o[F_OUT]) : wrap(y);
    if (!want_last && !want_ckpt) return py;
    PyObject *res = PyTuple_New(1 + want_last + want_ckpt);
    PyTuple_SET_ITEM(res, 0, py);
    if (want_last) PyTuple_SET_ITEM(res, 1, wrap(last));
    if (want_ckpt) PyTuple_SET_ITEM(res, 1 + want_last, wrap(ckpt));
    return res;
}

template <bool CPLX> PyObject *backward(PyObject *args, PyObject *kwargs) {
    PyObject *o[kMaxArgs];
    std::conditional_t<CPLX, lrnnx_ss_bwd_complex_args, lrnnx_ss_bwd_args> a = {};
    Call c;
    bool softplus, want_dx0;
    if (!c.good || !gather(kBwd, args, kwargs, o) || !disc_mode(o[B_DISC], a.disc) || !path_mode(o[B_PATH], a.path) ||
        !flag(o[B_SOFTPLUS], true, softplus) || !flag(o[B_DX0], false, want_dx0) || !absent(o[B_OUTS]) || !absent(o[B_WS]) ||
        !steps(o[B_LONGEST], a.max_seqlen)) Py_RETURN_NONE;
    a.delta_softplus = softplus;
    const at::Tensor *u = c.needed(o[B_U]), *delta = c.needed(o[B_DELTA]), *A = c.needed(o[B_A]), *Bm = c.needed(o[B_BM]), *Cm = c.needed(o[B_CM]);
    const at::Tensor *Dskip = c.tensor(o[B_D]), *bias = c.tensor(o[B_BIAS]), *z = c.tensor(o[B_Z]), *x0 = c.tensor(o[B_X0]);
    const at::Tensor *dy = c.needed(o[B_DY]), *ckpt = c.tensor(o[B_CKPT]);
    Scan s;
    s.read<CPLX>(c, a, o[B_CU], u, delta, A, Bm, Cm, Dskip, bias, z, x0);
    if (c.good) {
        c.rows(dy, s.io, s.rows, a.dy, a.dy_stride_b, a.dy_stride_d);
        c.data(ckpt, s.state, s.ckpt, a.ckpt);
    }
    if (!c.good) Py_RETURN_NONE;
    struct { const char *name; at::Tensor t; } outs[9];
    int n = 0;
    auto make = [&](const char *name, c10::IntArrayRef shape, c10::ScalarType type) -> const at::Tensor * {
        outs[n].name = name;
        outs[n].t = c.make(shape, type);
        return &outs[n++].t;
    };
    c.rows(make("du", s.rows, s.io), s.io, s.rows, a.du, a.du_stride_b, a.du_stride_d);
    c.rows(make("ddelta", s.rows, s.io), s.io, s.rows, a.ddelta, a.ddelta_stride_b, a.ddelta_stride_d);
    if (z) c.rows(make("dz", s.rows, s.io), s.io, s.rows, a.dz, a.dz_stride_b, a.dz_stride_d);
    c.data(make("dA", s.dn, s.state), s.state, s.dn, a.dA);
    c.data(make("dBm", s.one_map, s.state), s.state, s.one_map, a.dBm);
    c.data(make("dCm", s.one_map, s.state), s.state, s.one_map, a.dCm);
    if (Dskip) c.data(make("dD", s.d1, at::kFloat), at::kFloat, s.d1, a.dD);
    if (bias) c.data(make("dbias", s.d1, at::kFloat), at::kFloat, s.d1, a.dbias);
    if (want_dx0) c.data(make("dx0", s.bdn, s.state), s.state, s.bdn, a.dx0);
    size_t bytes;
    if constexpr (CPLX) {
        // with the forward's checkpoints only the chunk aggregates (or the launch order of a packed batch) and the sums of dBm and dCm
        bytes = lib.bytes(LRNNX_WS_BWD_COMPLEX, s.B, s.D, s.N, s.L, a.io_dtype, (int)s.G, s.packed);
        if (ckpt) bytes -= ((size_t)ckpt->numel() * 8 + 255) / 256 * 256;
    } else bytes = lib.bwd_bytes(&a);
    at::Tensor ws;
    if (bytes) ws = c.scratch(a, bytes);
    a.stream = c.stream();
    bool done;
    if constexpr (CPLX) done = launched(lib.cbwd, a); else done = launched(lib.bwd, a);
    if (!done) return nullptr;
    PyObject *res = PyDict_New();
    for (int i = 0; i < n; ++i) {
        PyObject *t = wrap(outs[i].t);
        PyDict_SetItemString(res, outs[i].name, t);
        Py_DECREF(t);
    }
    return res;
}

// one token, real or complex A
template <bool CPLX> PyObject *step(PyObject *args, PyObject *kwargs) {
    PyObject *o[kMaxArgs];
    std::conditional_t<CPLX, lrnnx_ss_step_complex_args, lrnnx_ss_step_args> a = {};
    Call c;
    bool softplus;
    if (!c.good || !gather(kStep, args, kwargs, o) || !disc_mode(o[9], a.disc) || !flag(o[10], true, softplus)) Py_RETURN_NONE;
    const at::Tensor *x = c.needed(o[0]), *u = c.needed(o[1]), *delta = c.needed(o[2]), *A = c.needed(o[3]), *Bm = c.needed(o[4]);
    const at::Tensor *Cm = c.needed(o[5]), *Dskip = c.tensor(o[6]), *bias = c.tensor(o[7]), *z = c.tensor(o[8]), *out = c.tensor(o[11]);
    if (!c.good || x->dim() != 3) Py_RETURN_NONE;
    const int64_t B = x->size(0), D = x->size(1), N = x->size(2);
    const c10::ScalarType io = u->scalar_type(), state = CPLX ? at::kComplexFloat : at::kFloat;
    const bool pairs = CPLX && io == at::kBFloat16;
    const c10::ScalarType map_type = CPLX && !pairs ? at::kComplexFloat : io;
    const Shape bd = {B, D}, dn = {D, N}, bdn = {B, D, N}, d1 = {D};
    Shape maps = {B};
    int64_t G = 1;
    if (Bm->dim() == 3 + pairs) maps.push_back(G = Bm->size(1));
    maps.push_back(N);
    if (pairs) maps.push_back(2);
    if ((io != at::kBFloat16 && io != at::kFloat) || G < 1 || D % G || !fits32(B) || !fits32(D) || !fits32(N)) Py_RETURN_NONE;
    a.struct_size = sizeof(a);
    a.B = (int32_t)B; a.D = (int32_t)D; a.N = (int32_t)N; a.bc_groups = (int32_t)G;
    a.io_dtype = io == at::kBFloat16 ? LRNNX_BF16 : LRNNX_F32;
    a.delta_softplus = softplus;
    c.data(x, state, bdn, a.x);
    // (the general path leaves the sizes of u, delta, z and out to its caller; only whole ones are taken here)
    c.row(u, io, bd, a.u, a.u_stride_b, a.u_stride_d);
    c.row(delta, io, bd, a.delta, a.delta_stride_b, a.delta_stride_d);
    c.row(z, io, bd, a.z, a.z_stride_b, a.z_stride_d);
    c.data(A, state, dn, a.A);
    c.data(Bm, map_type, maps, a.Bm);
    c.data(Cm, map_type, maps, a.Cm);
    c.data(Dskip, at::kFloat, d1, a.Dskip);
    c.data(bias, at::kFloat, d1, a.delta_bias);
    c.row(out, io, bd, a.y, a.y_stride_b, a.y_stride_d);
    if (!c.good) Py_RETURN_NONE;
    at::Tensor y;
    if (!out) {
        y = c.make(bd, io);
        c.row(&y, io, bd, a.y, a.y_stride_b, a.y_stride_d);
    }
    a.stream = c.stream();
    bool done;
    if constexpr (CPLX) done = launched(lib.cstep, a); else done = launched(lib.step, a);
    if (!done) return nullptr;
    return out ? given(o[11]) : wrap(y);
}

// x_k = lam x_{k-1} + v_k, and x_k = a_k x_{k-1} + b_k
template <bool LTI> PyObject *chain(PyObject *args, PyObject *kwargs) {
    PyObject *o[kMaxArgs];
    std::conditional_t<LTI, lrnnx_lti_args, lrnnx_diag_scan_args> a = {};
    Call c;
    bool want_last;
    if (!c.good || !gather(LTI ? kLti : kDiag, args, kwargs, o) || !flag(o[3], false, want_last) || !absent(o[5]) || !absent(o[LTI ? 7 : 6])) Py_RETURN_NONE;
    if constexpr (LTI) { if (!path_mode(o[6], a.path)) Py_RETURN_NONE; }
    const at::Tensor *m = c.needed(o[0]), *v = c.needed(o[1]), *x0 = c.tensor(o[2]), *out = c.tensor(o[4]);
    if (!c.good || v->dim() != 3) Py_RETURN_NONE;
    const int64_t B = v->size(0), L = v->size(1), P = v->size(2);
    const c10::ScalarType type = v->scalar_type();
    if ((type != at::kComplexFloat && (LTI || type != at::kFloat)) || !fits32(B) || !fits32(P)) Py_RETURN_NONE;
    const Shape blp = {B, L, P}, bp = {B, P}, p1 = {P};
    a.struct_size = sizeof(a);
    a.B = (int32_t)B; a.P = (int32_t)P; a.L = L;
    if constexpr (LTI) {
        c.data(m, type, p1, a.lambda);
        c.data(v, type, blp, a.v);
    } else {
        a.dtype = type == at::kFloat ? LRNNX_F32 : LRNNX_C64;
        c.data(m, type, blp, a.a);
        c.data(v, type, blp, a.b);
    }
    c.data(x0, type, bp, a.x0);
    c.data(out, type, blp, a.x);
    if (!c.good) Py_RETURN_NONE;
    at::Tensor x, last, ws;
    if (!out) { x = at::empty_like(*v); c.data(&x, type, blp, a.x); }
    if (want_last) { last = c.make(bp, type); c.data(&last, type, bp, a.x_last); }
    size_t bytes;
    if constexpr (LTI) bytes = lib.bytes(LRNNX_WS_LTI, B, P, 0, L, 0, 1, 0);
    else bytes = lib.bytes(LRNNX_WS_DIAG, B, P, 0, L, a.dtype, 1, 0);
    ws = c.scratch(a, std::max<size_t>(bytes, 16));
    a.stream = c.stream();
    bool done;
    if constexpr (LTI) done = launched(lib.lti, a); else done = launched(lib.diag, a);
    if (!done) return nullptr;
    PyObject *px = out ? given(o[4]) : wrap(x);
    if (!want_last) return px;
    PyObject *res = PyTuple_New(2);
    PyTuple_SET_ITEM(res, 0, px);
    PyTuple_SET_ITEM(res, 1, wrap(last));
    return res;
}

// their adjoints
template <bool LTI> PyObject *chain_bwd(PyObject *args, PyObject *kwargs) {
    PyObject *o[kMaxArgs];
    std::conditional_t<LTI, lrnnx_lti_bwd_args, lrnnx_diag_scan_bwd_args> a = {};
    Call c;
    bool want_dx0;
    if (!c.good || !gather(LTI ? kLtiBwd : kDiagBwd, args, kwargs, o) || !flag(o[4], true, want_dx0) || !absent(o[LTI ? 6 : 5]) ||
        !absent(o[LTI ? 7 : 6])) Py_RETURN_NONE;
    const at::Tensor *m = c.needed(o[0]), *x = c.needed(o[1]), *gx = c.needed(o[2]), *x0 = c.tensor(o[3]);
    const at::Tensor *out = LTI ? c.tensor(o[5]) : nullptr;
    if (!c.good || x->dim() != 3) Py_RETURN_NONE;
    const int64_t B = x->size(0), L = x->size(1), P = x->size(2);
    const c10::ScalarType type = x->scalar_type();
    if ((type != at::kComplexFloat && (LTI || type != at::kFloat)) || !fits32(B) || !fits32(P)) Py_RETURN_NONE;
    const Shape blp = {B, L, P}, bp = {B, P}, p1 = {P};
    a.struct_size = sizeof(a);
    a.B = (int32_t)B; a.P = (int32_t)P; a.L = L;
    if constexpr (LTI) c.data(m, type, p1, a.lambda);
    else {
        a.dtype = type == at::kFloat ? LRNNX_F32 : LRNNX_C64;
        c.data(m, type, blp, a.a);
    }
    c.data(x, type, blp, a.x);
    c.data(gx, type, blp, a.gx);
    c.data(x0, type, bp, a.x0);
    if constexpr (LTI) c.data(out, type, blp, a.dv);
    if (!c.good) Py_RETURN_NONE;
    at::Tensor first, second, dx0, ws;                   // dv and dlam, or da and db
    size_t bytes;
    if constexpr (LTI) {
        if (!out) { first = at::empty_like(*gx); c.data(&first, type, blp, a.dv); }
        second = c.make(p1, type); c.data(&second, type, p1, a.dlambda);
        bytes = lib.bytes(LRNNX_WS_LTI_BWD, B, P, 0, L, 0, 1, 0);
    } else {
        first = at::empty_like(*m); c.data(&first, type, blp, a.da);
        second = at::empty_like(*m); c.data(&second, type, blp, a.db);
        bytes = lib.bytes(LRNNX_WS_DIAG_BWD, B, P, 0, L, a.dtype, 1, 0);
    }
    if (want_dx0) { dx0 = c.make(bp, type); c.data(&dx0, type, bp, a.dx0); }
    ws = c.scratch(a, std::max<size_t>(bytes, 16));
    a.stream = c.stream();
    bool done;
    if constexpr (LTI) done = launched(lib.lti_bwd, a); else done = launched(lib.diag_bwd, a);
    if (!done) return nullptr;
    PyObject *res = PyTuple_New(3);
    PyTuple_SET_ITEM(res, 0, out ? given(o[5]) : wrap(first));
    PyTuple_SET_ITEM(res, 1, wrap(second));
    PyTuple_SET_ITEM(res, 2, want_dx0 ? wrap(dx0) : given(Py_None));
    return res;
}

template <PyObject *(*F)(PyObject *, PyObject *)> PyObject *entry(PyObject *, PyObject *const *p, Py_ssize_t n) {
    if (n != 2 || !PyTuple_CheckExact(p[0]) || !PyDict_CheckExact(p[1]) || !check_status) Py_RETURN_NONE;
    HANDLE_TH_ERRORS
    return F(p[0], p[1]);
    END_HANDLE_TH_ERRORS
}

// bind(check, interval, (addresses of the entry points in the order of `lib`))
PyObject *bind(PyObject *, PyObject *args) {
    PyObject *check, *addresses;
    long long interval;
    if (!PyArg_ParseTuple(args, "OLO!", &check, &interval, &PyTuple_Type, &addresses)) return nullptr;
    if (PyTuple_GET_SIZE(addresses) != kEntries) { PyErr_SetString(PyExc_ValueError, "bind: number of addresses"); return nullptr; }
    void *p[kEntries];
    for (int i = 0; i < kEntries; ++i) p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
    if (PyErr_Occurred()) return nullptr;
    std::memcpy(&lib, p, sizeof(lib));
    ckpt_interval = interval;
    Py_INCREF(check);
    Py_XDECREF(check_status);
    check_status = check;
    Py_RETURN_NONE;
}

PyMethodDef method(const char *name, PyObject *(*f)(PyObject *, PyObject *const *, Py_ssize_t)) {
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, "(args, kwargs) -> the call's result, or None: not taken"};
}
PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, "bind(check, interval, addresses of the entry points)"},
    method("lrnnx_selective_scan_fwd", entry<forward<false>>),
    method("lrnnx_selective_scan_bwd", entry<backward<false>>),
    method("lrnnx_selective_scan_fwd_complex", entry<forward<true>>),
    method("lrnnx_selective_scan_bwd_complex", entry<backward<true>>),
    method("lrnnx_selective_step", entry<step<false>>),
    method("lrnnx_selective_step_complex", entry<step<true>>),
    method("lrnnx_lti_diag_scan", entry<chain<true>>),
    method("lrnnx_lti_diag_scan_bwd", entry<chain_bwd<true>>),
    method("lrnnx_diag_scan", entry<chain<false>>),
    method("lrnnx_diag_scan_bwd", entry<chain_bwd<false>>),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "usual forms of the entry points' calls", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
    for (Names *n : {&kFwd, &kFwdComplex, &kBwd, &kStep, &kLti, &kLtiBwd, &kDiag, &kDiagBwd})
        for (int i = 0; i < n->count; ++i)
            if (!(n->key[i] = PyUnicode_InternFromString(n->text[i]))) return nullptr;
    return PyModule_Create(&module);
}
