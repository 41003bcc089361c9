// The host path of the binding for its ordinary calls: every argument a plain
// torch tensor of the documented type, shape and device, outputs not given, the
// current stream. A function here checks that, allocates the outputs as
// torch.empty does, makes the C call and returns the outputs as a tuple. It
// returns None, with nothing allocated or enqueued, where anything is otherwise
// (the caller's Python path then does what there is to do, or says what is
// wrong), and an int where a C call failed: its place in the chain << 8 | the
// status.
//
// Why native: policy_update took ~46 us of host time in Python (11 outputs, 25
// checks, three ctypes calls of up to 25 arguments) for kernels of 21 us at
// 512 x 4096 and 34 us at 96 x 152064.
#include <Python.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "dart.h"

namespace {

#define DART_FUNCTIONS(F)                                                        \
    F(dart_tok_stats) F(dart_tok_stats_ex) F(dart_select_tis_loss_fwd)           \
    F(dart_tis_grad) F(dart_tis_grad_ex) F(dart_grpo_advantage)                  \
    F(dart_step_select_groups) F(dart_tis_loss_fwd_ex)                           \
    F(dart_lmhead_tok_stats) F(dart_lmhead_tok_stats_ex)                         \
    F(dart_tis_loss_split_workspace_bytes) F(dart_lmhead_stats_workspace_bytes)

struct Lib {
#define DECLARE(name) decltype(&::name) name = nullptr;
    DART_FUNCTIONS(DECLARE)
#undef DECLARE
} lib;

using at::Tensor;

// The tensor behind an argument that is exactly a torch.Tensor (or a
// Parameter), strided and on a GPU; null for anything else.
const Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const Tensor& t = THPVariable_Unpack(o);
    return t.defined() && t.layout() == at::kStrided && t.is_cuda() ? &t : nullptr;
}

// A contiguous vector of n elements of the given type and device.
template <class T>
bool vec(PyObject* o, at::ScalarType type, int64_t n, at::Device dev, const T*& p) {
    const Tensor* t = plain(o);
    if (!t || t->scalar_type() != type || t->device() != dev || t->dim() != 1 ||
        t->numel() != n || !t->is_contiguous())
        return false;
    p = static_cast<const T*>(t->data_ptr());
    return true;
}

// A length of a 1-D tensor that some other check covers; -1 where there is none.
int64_t length(PyObject* o) {
    const Tensor* t = plain(o);
    return t && t->dim() == 1 ? t->numel() : -1;
}

bool number(PyObject* o, double& x) {
    if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) return false;
    x = PyFloat_AsDouble(o);
    if (x != -1.0 || !PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}

struct Logits {
    const Tensor* t;
    dart_dtype_t dtype;
    int64_t T, V, ld;
    at::Device dev{at::kCPU};
};

bool logits(PyObject* o, Logits& z) {
    z.t = plain(o);
    if (!z.t || z.t->dim() != 2 || z.t->stride(1) != 1) return false;
    if (z.t->scalar_type() == at::kBFloat16)
        z.dtype = DART_BF16;
    else if (z.t->scalar_type() == at::kFloat)
        z.dtype = DART_F32;
    else
        return false;
    z.T = z.t->size(0), z.V = z.t->size(1), z.ld = z.t->stride(0), z.dev = z.t->device();
    return true;
}

Tensor empty(at::IntArrayRef size, at::ScalarType type, at::Device dev) {
    return at::empty(size, at::TensorOptions().dtype(type).device(dev));
}

hipStream_t stream_of(at::Device dev) {
    return c10::hip::getCurrentHIPStream(dev.index()).stream();
}

float* f32(const Tensor& t) { return static_cast<float*>(t.data_ptr()); }
double* f64(const Tensor& t) { return static_cast<double*>(t.data_ptr()); }
int32_t* i32(const Tensor& t) { return static_cast<int32_t*>(t.data_ptr()); }
uint8_t* u8(const Tensor& t) { return static_cast<uint8_t*>(t.data_ptr()); }

// f() without the interpreter lock, as ctypes calls it.
template <class F>
dart_status_t call(F&& f) {
    dart_status_t st;
    Py_BEGIN_ALLOW_THREADS;
    st = f();
    Py_END_ALLOW_THREADS;
    return st;
}

PyObject* failed(int place, dart_status_t st) { return PyLong_FromLong(place << 8 | (int)st); }

template <class... Ts>
PyObject* tuple(const Ts&... ts) {
    PyObject* out = PyTuple_New(sizeof...(ts));
    if (!out) return nullptr;
    Py_ssize_t i = 0;
    auto put = [&](const Tensor& t) {
        PyObject* o = Py_None;
        if (t.defined())
            o = THPVariable_Wrap(t);
        else
            Py_INCREF(o);
        PyTuple_SET_ITEM(out, i++, o);
        return o != nullptr;
    };
    if ((put(ts) && ...)) return out;
    Py_DECREF(out);
    return nullptr;
}

struct TokStats {
    Tensor logp, entropy, lse;
    TokStats(int64_t T, at::Device dev)
        : logp(empty({T}, at::kFloat, dev)),
          entropy(empty({T}, at::kFloat, dev)),
          lse(empty({T}, at::kFloat, dev)) {}
};

dart_status_t run_tok_stats(const Logits& z, const int32_t* y, double inv_temp, const TokStats& s,
                            hipStream_t st) {
    const void* p = z.t->data_ptr();
    return call([&] {
        return inv_temp == 1.0
                   ? lib.dart_tok_stats(p, z.dtype, z.T, z.V, z.ld, y, f32(s.logp), f32(s.entropy),
                                        f32(s.lse), st)
                   : lib.dart_tok_stats_ex(p, z.dtype, z.T, z.V, z.ld, y, (float)inv_temp,
                                           f32(s.logp), f32(s.entropy), f32(s.lse), st);
    });
}

struct SelectLoss {
    int64_t T = 0, S = 0;
    const float *entropy = nullptr, *logp = nullptr, *old = nullptr, *roll = nullptr,
                *adv = nullptr;
    const int32_t* off = nullptr;
    double rho, eps_low, eps_high, C;
    Tensor step_entropy, step_mask, n_kept, loss, coef, stats, workspace;

    // logp_old, logp_rollout, adv, step_offsets, rho, eps_low, eps_high, C
    bool take(PyObject* const* a, int64_t T_, at::Device dev) {
        T = T_, S = length(a[3]) - 1;
        return S >= 0 && vec(a[0], at::kFloat, T, dev, old) && vec(a[1], at::kFloat, T, dev, roll) &&
               vec(a[2], at::kFloat, T, dev, adv) && vec(a[3], at::kInt, S + 1, dev, off) &&
               number(a[4], rho) && number(a[5], eps_low) && number(a[6], eps_high) &&
               number(a[7], C);
    }
    dart_status_t run(at::Device dev, bool with_stats, hipStream_t st) {
        step_entropy = empty({S}, at::kFloat, dev), step_mask = empty({S}, at::kByte, dev);
        n_kept = empty({1}, at::kInt, dev), loss = empty({1}, at::kDouble, dev);
        coef = empty({T}, at::kFloat, dev);
        if (with_stats) stats = empty({4}, at::kFloat, dev);
        const size_t bytes = lib.dart_tis_loss_split_workspace_bytes(T);
        workspace = empty({(int64_t)bytes}, at::kByte, dev);
        return call([&] {
            return lib.dart_select_tis_loss_fwd(
                T, entropy, logp, old, roll, adv, off, S, rho, (float)eps_low, (float)eps_high,
                (float)C, f32(step_entropy), u8(step_mask), i32(n_kept), f64(loss), f32(coef),
                stats.defined() ? f32(stats) : nullptr, workspace.data_ptr(), bytes, st);
        });
    }
};

// dlogits given (checked) or made.
bool take_dlogits(PyObject* o, const Logits& z, Tensor& dz) {
    if (o == Py_None) return true;
    const Tensor* t = plain(o);
    if (!t || t->scalar_type() != z.t->scalar_type() || t->dim() != 2 || t->size(0) != z.T ||
        t->size(1) != z.V || t->stride(1) != 1 || t->device() != z.dev)
        return false;
    dz = *t;
    return true;
}

dart_status_t run_grad(const Logits& z, const int32_t* y, const float* logp, const float* lse,
                       const float* coef, double inv_temp, bool skip, Tensor& dz, hipStream_t st) {
    if (!dz.defined()) dz = empty({z.T, z.V}, z.t->scalar_type(), z.dev);
    const void* p = z.t->data_ptr();
    void* q = dz.data_ptr();
    const int64_t ld = dz.stride(0);
    return call([&] {
        return inv_temp == 1.0 && !skip
                   ? lib.dart_tis_grad(p, z.dtype, z.T, z.V, z.ld, y, logp, lse, coef, q, ld, st)
                   : lib.dart_tis_grad_ex(p, z.dtype, z.T, z.V, z.ld, y, logp, lse, coef,
                                          (float)inv_temp, skip ? DART_GRAD_SKIP_ZERO_ROWS : 0u, q,
                                          ld, st);
    });
}

// ---------------------------------------------------------------------------
// the module's functions
// ---------------------------------------------------------------------------

#define NATIVE(name, nargs)                                                    \
    PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n) {              \
        HANDLE_TH_ERRORS                                                       \
        if (n != nargs) {                                                      \
            PyErr_SetString(PyExc_TypeError, #name ": wrong argument count");  \
            return nullptr;                                                    \
        }

#define NATIVE_END \
    END_HANDLE_TH_ERRORS \
    }

// logits, target, inv_temp
NATIVE(tok_stats, 3)
    Logits z;
    const int32_t* y;
    double it;
    if (!logits(a[0], z) || !vec(a[1], at::kInt, z.T, z.dev, y) || !number(a[2], it)) Py_RETURN_NONE;
    TokStats s(z.T, z.dev);
    if (const dart_status_t st = run_tok_stats(z, y, it, s, stream_of(z.dev)); st != DART_OK)
        return failed(it == 1.0 ? 0 : 1, st);
    return tuple(s.logp, s.entropy, s.lse);
NATIVE_END

// entropy, logp, logp_old, logp_rollout, adv, step_offsets, rho, eps_low, eps_high, C, with_stats
NATIVE(select_tis_loss_fwd, 11)
    const Tensor* lp = plain(a[1]);
    SelectLoss x;
    if (!lp || lp->dim() != 1) Py_RETURN_NONE;
    const at::Device dev = lp->device();
    const int64_t T = lp->numel();
    if (!vec(a[0], at::kFloat, T, dev, x.entropy) || !vec(a[1], at::kFloat, T, dev, x.logp) ||
        !x.take(a + 2, T, dev))
        Py_RETURN_NONE;
    if (const dart_status_t st = x.run(dev, a[10] == Py_True, stream_of(dev)); st != DART_OK)
        return failed(0, st);
    return tuple(x.step_entropy, x.step_mask, x.n_kept, x.loss, x.coef, x.stats);
NATIVE_END

// logits, target, logp, lse, tok_coef, dlogits, inv_temp, skip_zero_rows
NATIVE(tis_grad, 8)
    Logits z;
    const int32_t* y;
    const float *logp, *lse, *coef;
    double it;
    Tensor dz;
    if (!logits(a[0], z) || !vec(a[1], at::kInt, z.T, z.dev, y) ||
        !vec(a[2], at::kFloat, z.T, z.dev, logp) || !vec(a[3], at::kFloat, z.T, z.dev, lse) ||
        !vec(a[4], at::kFloat, z.T, z.dev, coef) || !take_dlogits(a[5], z, dz) ||
        !number(a[6], it) || !PyBool_Check(a[7]))
        Py_RETURN_NONE;
    const bool skip = a[7] == Py_True;
    const dart_status_t st = run_grad(z, y, logp, lse, coef, it, skip, dz, stream_of(z.dev));
    if (st != DART_OK) return failed(it == 1.0 && !skip ? 0 : 1, st);
    if (a[5] != Py_None) {
        Py_INCREF(a[5]);
        return a[5];
    }
    return THPVariable_Wrap(dz);
NATIVE_END

// logits, target, logp_old, logp_rollout, adv, step_offsets, rho, eps_low, eps_high, C, dlogits
NATIVE(policy_update, 11)
    Logits z;
    const int32_t* y;
    SelectLoss x;
    Tensor dz;
    if (!logits(a[0], z) || !vec(a[1], at::kInt, z.T, z.dev, y) || !x.take(a + 2, z.T, z.dev) ||
        !take_dlogits(a[10], z, dz))
        Py_RETURN_NONE;
    const hipStream_t s = stream_of(z.dev);
    TokStats ts(z.T, z.dev);
    if (const dart_status_t st = run_tok_stats(z, y, 1.0, ts, s); st != DART_OK)
        return failed(0, st);
    x.entropy = f32(ts.entropy), x.logp = f32(ts.logp);
    if (const dart_status_t st = x.run(z.dev, true, s); st != DART_OK) return failed(1, st);
    if (const dart_status_t st =
            run_grad(z, y, x.logp, f32(ts.lse), f32(x.coef), 1.0, false, dz, s);
        st != DART_OK)
        return failed(2, st);
    return tuple(ts.logp, ts.entropy, ts.lse, x.step_entropy, x.step_mask, x.n_kept, x.loss, dz,
                 x.coef, x.stats);
NATIVE_END

// reward, traj_step_offsets, group_traj_offsets, step_offsets, T
NATIVE(grpo_advantage, 5)
    const Tensor* r = plain(a[0]);
    if (!r || r->dim() != 1 || !PyLong_CheckExact(a[4])) Py_RETURN_NONE;
    const at::Device dev = r->device();
    const int64_t n = r->numel(), G = length(a[2]) - 1, S = length(a[3]) - 1;
    const float* reward;
    const int32_t *traj, *grp, *off;
    const int64_t T = PyLong_AsLongLong(a[4]);
    if (T < 1 || G < 0 || S < 0 || !vec(a[0], at::kFloat, n, dev, reward) ||
        !vec(a[1], at::kInt, n + 1, dev, traj) || !vec(a[2], at::kInt, G + 1, dev, grp) ||
        !vec(a[3], at::kInt, S + 1, dev, off)) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const Tensor adv = empty({T}, at::kFloat, dev), mean = empty({G}, at::kFloat, dev),
                 sd = empty({G}, at::kFloat, dev);
    const hipStream_t s = stream_of(dev);
    const dart_status_t st = call([&] {
        return lib.dart_grpo_advantage(reward, n, traj, grp, G, off, S, T, f32(adv), f32(mean),
                                       f32(sd), s);
    });
    return st == DART_OK ? tuple(adv, mean, sd) : failed(0, st);
NATIVE_END

// entropy, step_offsets, group_step_offsets, rho
NATIVE(step_select_groups, 4)
    const Tensor* e = plain(a[0]);
    double rho;
    if (!e || e->dim() != 1 || !number(a[3], rho)) Py_RETURN_NONE;
    const at::Device dev = e->device();
    const int64_t T = e->numel(), S = length(a[1]) - 1, G = length(a[2]) - 1;
    const float* entropy;
    const int32_t *off, *grp;
    if (S < 0 || G < 0 || !vec(a[0], at::kFloat, T, dev, entropy) ||
        !vec(a[1], at::kInt, S + 1, dev, off) || !vec(a[2], at::kInt, G + 1, dev, grp))
        Py_RETURN_NONE;
    const Tensor ent = empty({S}, at::kFloat, dev), mask = empty({S}, at::kByte, dev),
                 kept = empty({G}, at::kInt, dev);
    const hipStream_t s = stream_of(dev);
    const dart_status_t st = call([&] {
        return lib.dart_step_select_groups(entropy, T, off, S, grp, G, rho, f32(ent), u8(mask),
                                           i32(kept), s);
    });
    return st == DART_OK ? tuple(ent, mask, kept) : failed(0, st);
NATIVE_END

// logp, logp_old, logp_rollout, adv, step_offsets, step_mask, logp_ref, eps_low, eps_high, C, kl,
// beta, aggregation, ratio, with_stats
NATIVE(tis_loss_fwd_ex, 15)
    const Tensor* lp = plain(a[0]);
    if (!lp || lp->dim() != 1) Py_RETURN_NONE;
    const at::Device dev = lp->device();
    const int64_t T = lp->numel(), S = length(a[4]) - 1;
    const float *logp, *old, *roll, *adv, *ref = nullptr;
    const int32_t* off;
    const uint8_t* mask;
    double v[7];
    for (int i = 0; i < 7; ++i)
        if (!number(a[7 + i], v[i])) Py_RETURN_NONE;
    const bool with_kl = v[3] != 0;
    if (S < 0 || !vec(a[0], at::kFloat, T, dev, logp) || !vec(a[1], at::kFloat, T, dev, old) ||
        !vec(a[2], at::kFloat, T, dev, roll) || !vec(a[3], at::kFloat, T, dev, adv) ||
        !vec(a[4], at::kInt, S + 1, dev, off) || !vec(a[5], at::kByte, S, dev, mask) ||
        (with_kl && !vec(a[6], at::kFloat, T, dev, ref)))
        Py_RETURN_NONE;
    dart_loss_config_t cfg;
    cfg.eps_low = (float)v[0], cfg.eps_high = (float)v[1], cfg.C = (float)v[2];
    cfg.kl = static_cast<decltype(cfg.kl)>((int)v[3]);
    cfg.beta = (float)v[4];
    cfg.aggregation = static_cast<decltype(cfg.aggregation)>((int)v[5]);
    cfg.ratio = static_cast<decltype(cfg.ratio)>((int)v[6]);
    const Tensor loss = empty({1}, at::kDouble, dev), coef = empty({T}, at::kFloat, dev);
    Tensor stats;
    if (a[14] == Py_True) stats = empty({6}, at::kFloat, dev);
    const size_t bytes = lib.dart_tis_loss_split_workspace_bytes(T);
    const Tensor ws = empty({(int64_t)bytes}, at::kByte, dev);
    const hipStream_t s = stream_of(dev);
    const dart_status_t st = call([&] {
        return lib.dart_tis_loss_fwd_ex(T, logp, old, roll, ref, adv, off, S, mask, &cfg, f64(loss),
                                        f32(coef), stats.defined() ? f32(stats) : nullptr,
                                        ws.data_ptr(), bytes, s);
    });
    return st == DART_OK ? tuple(loss, coef, stats) : failed(0, st);
NATIVE_END

bool matrix(PyObject* o, const Tensor*& t) {
    t = plain(o);
    return t && t->scalar_type() == at::kBFloat16 && t->dim() == 2 && t->stride(1) == 1 &&
           t->stride(0) % 8 == 0 && reinterpret_cast<uintptr_t>(t->data_ptr()) % 16 == 0;
}

// hidden, weight, target, inv_temp (None: the call without one)
NATIVE(lmhead_tok_stats, 4)
    const Tensor *h, *w;
    const int32_t* y;
    double it = 1.0;
    const bool ex = a[3] != Py_None;
    if (!matrix(a[0], h) || !matrix(a[1], w) || w->device() != h->device() ||
        w->size(1) != h->size(1) || !vec(a[2], at::kInt, h->size(0), h->device(), y) ||
        (ex && !number(a[3], it)))
        Py_RETURN_NONE;
    const at::Device dev = h->device();
    const int64_t T = h->size(0), d = h->size(1), V = w->size(0), ldh = h->stride(0),
                  ldw = w->stride(0);
    const TokStats o(T, dev);
    const size_t bytes = lib.dart_lmhead_stats_workspace_bytes(T, V);
    const Tensor ws = empty({(int64_t)bytes}, at::kByte, dev);
    const void *hp = h->data_ptr(), *wp = w->data_ptr();
    const hipStream_t s = stream_of(dev);
    const dart_status_t st = call([&] {
        return ex ? lib.dart_lmhead_tok_stats_ex(hp, T, d, ldh, wp, V, ldw, y, (float)it,
                                                 f32(o.logp), f32(o.entropy), f32(o.lse),
                                                 ws.data_ptr(), bytes, s)
                  : lib.dart_lmhead_tok_stats(hp, T, d, ldh, wp, V, ldw, y, f32(o.logp),
                                              f32(o.entropy), f32(o.lse), ws.data_ptr(), bytes, s);
    });
    return st == DART_OK ? tuple(o.logp, o.entropy, o.lse) : failed(0, st);
NATIVE_END

// open(path): the C functions of the library at path.
PyObject* open_lib(PyObject*, PyObject* arg) {
    const char* path = PyUnicode_AsUTF8(arg);
    if (!path) return nullptr;
    void* h = dlopen(path, RTLD_NOW | RTLD_LOCAL);
#define RESOLVE(name)                                                           \
    if (h && !(lib.name = reinterpret_cast<decltype(lib.name)>(dlsym(h, #name)))) h = nullptr;
    DART_FUNCTIONS(RESOLVE)
#undef RESOLVE
    if (!h) {
        PyErr_Format(PyExc_RuntimeError, "%s does not open or is not built from this source", path);
        return nullptr;
    }
    Py_RETURN_NONE;
}

#define ENTRY(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    ENTRY(tok_stats), ENTRY(select_tis_loss_fwd), ENTRY(tis_grad), ENTRY(policy_update),
    ENTRY(grpo_advantage), ENTRY(step_select_groups), ENTRY(tis_loss_fwd_ex),
    ENTRY(lmhead_tok_stats), {"open", open_lib, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods,
                          nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module_def); }
