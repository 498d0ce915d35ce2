// Native half of the Python binding: argument checks, output allocation and the C call of the entry points in one
// step.  A pass at the small shapes is a handful of kernels of 2-5 us each, and marshalling it in Python (attribute
// checks of a dozen tensors, an allocation per output, the current stream, ctypes conversions) took 12-15 us per call, as
// long as the kernels ran.  Measured per call, host time: lambda-return and its gradient 24.7 -> 8.7 us, one ssm_step
// 17.3 -> 7.8 us, forward of a 2 x 64 x 32 x 32 layer (three launches then) 29.3 -> 14.3 us; about 3 us of it per kernel launch either way.
//
// Contract with binding.py: every function takes positional arguments only and returns
//   the outputs (a tensor, a tuple or a dict) when the call was made and succeeded,
//   an int (the ssm_status) when the library refused it,
//   None when an argument is not what this half handles: binding.py then takes its general path, which does the
//   same checks one by one and raises the error that names the argument.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/ssm.h"

namespace {

constexpr auto F32 = c10::kFloat;
constexpr auto C64 = c10::kComplexFloat;
constexpr auto U8 = c10::kByte;

// One tensor argument.  ok: absent where that is allowed, or a contiguous GPU tensor of the type and shape wanted.
struct Arg {
    const at::Tensor *t = nullptr;
    bool none = false, bad = false;
    explicit Arg(PyObject *o)
    {
        if (o == Py_None) none = true;
        else if (THPVariable_Check(o)) t = &THPVariable_Unpack(o);
        else bad = true;
    }
    bool is(c10::ScalarType dt, std::initializer_list<int64_t> shape, bool optional = false) const
    {
        if (none) return optional;
        return !bad && t->is_cuda() && t->scalar_type() == dt && t->sizes() == c10::IntArrayRef(shape.begin(), shape.size()) &&
               t->is_contiguous();
    }
    int64_t dim() const { return t ? t->dim() : -1; }
    int64_t size(int i) const { return t->size(i); }
    template <class T> T *ptr() const { return t ? static_cast<T *>(t->data_ptr()) : nullptr; }
    const ssm_c64 *c64() const { return ptr<const ssm_c64>(); }
    const float *f32() const { return ptr<const float>(); }
    const uint8_t *u8() const { return ptr<const uint8_t>(); }
};

at::Tensor empty(std::initializer_list<int64_t> shape, c10::ScalarType dt, const at::Tensor &like)
{
    return at::Tensor(at::detail::empty_cuda(c10::IntArrayRef(shape.begin(), shape.size()), dt, like.device(), std::nullopt));
}
template <class T> T *raw(const at::Tensor &t) { return t.defined() ? static_cast<T *>(t.data_ptr()) : nullptr; }
ssm_c64 *c64(const at::Tensor &t) { return raw<ssm_c64>(t); }
float *f32(const at::Tensor &t) { return raw<float>(t); }

// An output: the caller's tensor when there is one, else a new one when it is wanted.
at::Tensor output(PyObject *given, bool wanted, std::initializer_list<int64_t> shape, c10::ScalarType dt, const at::Tensor &like, bool &bad)
{
    if (given && given != Py_None) {
        if (!THPVariable_Check(given)) { bad = true; return at::Tensor(); }
        return THPVariable_Unpack(given);
    }
    return wanted ? empty(shape, dt, like) : at::Tensor();
}

// The workspace: the caller's, or one of n bytes that lives until the call returns (its kernels are queued on the
// stream it was allocated on, so the allocator hands the block out again behind them).
struct Workspace {
    at::Tensor own;
    void *p = nullptr;
    size_t n = 0;
    bool bad = false;
    Workspace(const Arg &given, size_t need, const at::Tensor &like)
    {
        if (given.none) {
            if (need == 0) { bad = true; return; }
            own = empty({(int64_t)need}, U8, like);
            p = own.data_ptr(); n = need;
        } else if (given.t) {
            p = given.t->data_ptr(); n = (size_t)given.t->numel();
        } else {
            bad = true;
        }
    }
};

// Raw handle of the stream: the one given (an int), or the current one.  A workspace of this call's own is only
// allocated for the current stream.
bool stream_of(PyObject *o, const Arg *workspace, void *&s)
{
    if (o == Py_None) { s = c10::hip::getCurrentHIPStream().stream(); return true; }
    if (workspace && workspace->none) return false;
    s = PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}
bool yes(PyObject *o)
{
    if (o == Py_True || o == Py_False) return o == Py_True;
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw python_error();                 // (its error is the caller's)
    return v > 0;
}

PyObject *wrap(const at::Tensor &t)
{
    if (!t.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(t);
}
struct Named { const char *name; const at::Tensor *t; };
PyObject *dict(std::initializer_list<Named> items)
{
    PyObject *d = PyDict_New();
    for (const Named &i : items) {
        PyObject *v = wrap(*i.t);
        PyDict_SetItemString(d, i.name, v);
        Py_DECREF(v);
    }
    return d;
}
PyObject *tuple(std::initializer_list<const at::Tensor *> items)
{
    PyObject *r = PyTuple_New((Py_ssize_t)items.size());
    Py_ssize_t k = 0;
    for (const at::Tensor *t : items) PyTuple_SET_ITEM(r, k++, wrap(*t));
    return r;
}
PyObject *item(PyObject *d, const char *key) { return d == Py_None ? nullptr : PyDict_GetItemString(d, key); }

// The C call without the interpreter's lock.  Its arguments are values by then: taking a tensor's data pointer can throw (a
// tensor without storage, for instance a batched one), and an exception must find the lock held.
template <class... P, class... A>
ssm_status call_without_gil(ssm_status (*entry)(P...), A... args)
{
    static_assert(sizeof...(P) == sizeof...(A) && (std::is_trivially_copyable_v<A> && ...), "pointers and numbers");
    ssm_status rc;
    Py_BEGIN_ALLOW_THREADS
    rc = entry(args...);
    Py_END_ALLOW_THREADS
    return rc;
}

#define GENERAL_PATH_UNLESS(cond) do { if (!(cond)) Py_RETURN_NONE; } while (0)
#define CALL(...) \
    const ssm_status rc = call_without_gil(__VA_ARGS__); \
    if (rc != SSM_OK) return PyLong_FromLong((long)rc)
#define ENTRY(name) PyObject *name(PyObject *, PyObject *const *a, Py_ssize_t n)
// (torch's own translation: an allocation that fails raises torch.OutOfMemoryError here as on the general path)
#define TRY_BEGIN HANDLE_TH_ERRORS
#define TRY_END END_HANDLE_TH_ERRORS

// The eight inputs that the layer's calls share, and the shape they agree on.
struct LayerArgs {
    Arg Lambda, B, C, D, log_delta, u, is_first, x0;
    int64_t Bt = 0, L = 0, H = 0, P = 0;
    bool ok;
    explicit LayerArgs(PyObject *const *a)
        : Lambda(a[0]), B(a[1]), C(a[2]), D(a[3]), log_delta(a[4]), u(a[5]), is_first(a[6]), x0(a[7])
    {
        ok = u.dim() == 3 && Lambda.dim() == 1;
        if (!ok) return;
        Bt = u.size(0); L = u.size(1); H = u.size(2); P = Lambda.size(0);
        ok = Lambda.is(C64, {P}) && B.is(C64, {P, H}) && C.is(C64, {H, P}) && D.is(F32, {H}) && log_delta.is(F32, {P}) &&
             u.is(F32, {Bt, L, H}) && is_first.is(U8, {Bt, L}, true) && x0.is(C64, {Bt, P}, true);
    }
};

// (Lambda, B, C, D, log_delta, u, is_first, x0, want_x, want_x_last, workspace, stream, out)
ENTRY(scan_fwd)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 13);
    LayerArgs i(a);
    Arg ws(a[10]);
    void *s;
    GENERAL_PATH_UNLESS(i.ok && stream_of(a[11], &ws, s) && (a[12] == Py_None || PyDict_Check(a[12])));
    const at::Tensor &u = *i.u.t;
    Workspace w(ws, ws.none ? ssm_workspace_bytes(i.Bt, i.L, i.H, i.P, 0) : 0, u);
    bool bad = w.bad;
    at::Tensor y = output(item(a[12], "y"), true, {i.Bt, i.L, i.H}, F32, u, bad);
    at::Tensor x = output(item(a[12], "x"), yes(a[8]), {i.Bt, i.L, i.P}, C64, u, bad);
    at::Tensor xl = output(item(a[12], "x_last"), yes(a[9]), {i.Bt, i.P}, C64, u, bad);
    GENERAL_PATH_UNLESS(!bad);
    CALL(ssm_scan_fwd, i.Lambda.c64(), i.B.c64(), i.C.c64(), i.D.f32(), i.log_delta.f32(), i.u.f32(), i.is_first.u8(), i.x0.c64(),
                      i.Bt, i.L, i.H, i.P, f32(y), c64(x), c64(xl), w.p, w.n, s);
    return dict({{"y", &y}, {"x", &x}, {"x_last", &xl}});
    TRY_END
}

// (Lambda, B, C, D, log_delta, u, is_first, x0, x, dy, want_dx0, workspace, stream, out)
ENTRY(scan_bwd)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 14);
    LayerArgs i(a);
    Arg x(a[8]), dy(a[9]), ws(a[11]);
    void *s;
    GENERAL_PATH_UNLESS(i.ok && x.is(C64, {i.Bt, i.L, i.P}) && dy.is(F32, {i.Bt, i.L, i.H}) && stream_of(a[12], &ws, s) &&
                        (a[13] == Py_None || PyDict_Check(a[13])));
    const at::Tensor &u = *i.u.t;
    Workspace w(ws, ws.none ? ssm_workspace_bytes(i.Bt, i.L, i.H, i.P, 1) : 0, u);
    bool bad = w.bad;
    at::Tensor du = output(item(a[13], "du"), true, {i.Bt, i.L, i.H}, F32, u, bad);
    at::Tensor dL = output(item(a[13], "dLambda"), true, {i.P}, C64, u, bad);
    at::Tensor dB = output(item(a[13], "dB"), true, {i.P, i.H}, C64, u, bad);
    at::Tensor dC = output(item(a[13], "dC"), true, {i.H, i.P}, C64, u, bad);
    at::Tensor dD = output(item(a[13], "dD"), true, {i.H}, F32, u, bad);
    at::Tensor dl = output(item(a[13], "dlog_delta"), true, {i.P}, F32, u, bad);
    at::Tensor dx0 = output(item(a[13], "dx0"), yes(a[10]), {i.Bt, i.P}, C64, u, bad);
    GENERAL_PATH_UNLESS(!bad);
    CALL(ssm_scan_bwd, i.Lambda.c64(), i.B.c64(), i.C.c64(), i.D.f32(), i.log_delta.f32(), i.u.f32(), i.is_first.u8(), i.x0.c64(),
                      i.Bt, i.L, i.H, i.P, x.c64(), dy.f32(), f32(du), c64(dL), c64(dB), c64(dC), f32(dD), f32(dl), c64(dx0),
                      w.p, w.n, s);
    return dict({{"du", &du}, {"dLambda", &dL}, {"dB", &dB}, {"dC", &dC}, {"dD", &dD}, {"dlog_delta", &dl}, {"dx0", &dx0}});
    TRY_END
}

// (Lambda, B, C, D, log_delta, u, is_first, x0, W, want_gate, workspace, stream)
ENTRY(block_fwd)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 12);
    LayerArgs i(a);
    Arg W(a[8]), ws(a[10]);
    void *s;
    GENERAL_PATH_UNLESS(i.ok && W.is(F32, {i.H, i.H}) && stream_of(a[11], &ws, s));
    const at::Tensor &u = *i.u.t;
    Workspace w(ws, ws.none ? ssm_block_workspace_bytes(i.Bt, i.L, i.H, i.P, 0) : 0, u);
    GENERAL_PATH_UNLESS(!w.bad);
    at::Tensor y = empty({i.Bt, i.L, i.H}, F32, u), out = empty({i.Bt, i.L, i.H}, F32, u), gate;
    if (yes(a[9])) gate = empty({i.Bt, i.L, i.H}, F32, u);
    at::Tensor x = empty({i.Bt, i.L, i.P}, C64, u), xl = empty({i.Bt, i.P}, C64, u);
    CALL(ssm_block_fwd, i.Lambda.c64(), i.B.c64(), i.C.c64(), i.D.f32(), i.log_delta.f32(), W.f32(), i.u.f32(), i.is_first.u8(),
                       i.x0.c64(), i.Bt, i.L, i.H, i.P, f32(y), f32(out), f32(gate), c64(x), c64(xl), w.p, w.n, s);
    return dict({{"y", &y}, {"out", &out}, {"gate", &gate}, {"x", &x}, {"x_last", &xl}});
    TRY_END
}

// (Lambda, B, C, D, log_delta, u, is_first, x0, W, x, y, gate, dout, workspace, stream)
ENTRY(block_bwd)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 15);
    LayerArgs i(a);
    Arg W(a[8]), x(a[9]), y(a[10]), gate(a[11]), dout(a[12]), ws(a[13]);
    void *s;
    GENERAL_PATH_UNLESS(i.ok && W.is(F32, {i.H, i.H}) && x.is(C64, {i.Bt, i.L, i.P}) && y.is(F32, {i.Bt, i.L, i.H}) &&
                        gate.is(F32, {i.Bt, i.L, i.H}) && dout.is(F32, {i.Bt, i.L, i.H}) && stream_of(a[14], &ws, s));
    const at::Tensor &u = *i.u.t;
    Workspace w(ws, ws.none ? ssm_block_workspace_bytes(i.Bt, i.L, i.H, i.P, 1) : 0, u);
    GENERAL_PATH_UNLESS(!w.bad);
    at::Tensor du = empty({i.Bt, i.L, i.H}, F32, u), dL = empty({i.P}, C64, u), dB = empty({i.P, i.H}, C64, u),
               dC = empty({i.H, i.P}, C64, u), dD = empty({i.H}, F32, u), dl = empty({i.P}, F32, u), dx0 = empty({i.Bt, i.P}, C64, u),
               dW = empty({i.H, i.H}, F32, u);
    CALL(ssm_block_bwd, i.Lambda.c64(), i.B.c64(), i.C.c64(), i.D.f32(), i.log_delta.f32(), W.f32(), i.u.f32(), i.is_first.u8(),
                       i.x0.c64(), i.Bt, i.L, i.H, i.P, x.c64(), y.f32(), gate.f32(), dout.f32(), f32(du), c64(dL), c64(dB), c64(dC),
                       f32(dD), f32(dl), c64(dx0), f32(dW), w.p, w.n, s);
    return dict({{"du", &du}, {"dLambda", &dL}, {"dB", &dB}, {"dC", &dC}, {"dD", &dD}, {"dlog_delta", &dl}, {"dx0", &dx0}, {"dW", &dW}});
    TRY_END
}

// (Lambda, B, C, log_delta, stream)
ENTRY(step_prepare)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 5);
    Arg Lambda(a[0]), B(a[1]), C(a[2]), log_delta(a[3]);
    void *s;
    GENERAL_PATH_UNLESS(B.dim() == 2 && stream_of(a[4], nullptr, s));
    const int64_t P = B.size(0), H = B.size(1);
    GENERAL_PATH_UNLESS(Lambda.is(C64, {P}) && B.is(C64, {P, H}) && C.is(C64, {H, P}) && log_delta.is(F32, {P}));
    const size_t bytes = ssm_step_plan_bytes(H, P);
    GENERAL_PATH_UNLESS(bytes > 0);
    at::Tensor plan = empty({(int64_t)bytes}, U8, *B.t);
    CALL(ssm_step_prepare, Lambda.c64(), B.c64(), C.c64(), log_delta.f32(), H, P, plan.data_ptr(), bytes, s);
    return wrap(plan);
    TRY_END
}

// (plan, D, u, x_prev, is_first, P, x, y, stream)
ENTRY(step)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 9);
    Arg plan(a[0]), D(a[1]), u(a[2]), x_prev(a[3]), first(a[4]), xo(a[6]), yo(a[7]);
    void *s;
    GENERAL_PATH_UNLESS(plan.t && u.dim() == 2 && stream_of(a[8], nullptr, s) && !xo.bad && !yo.bad);
    const int64_t Bt = u.size(0), H = u.size(1);
    int64_t P;
    if (a[5] != Py_None) {
        P = PyLong_AsLongLong(a[5]);
        if (P == -1 && PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    } else {
        const Arg &from = x_prev.none ? xo : x_prev;
        GENERAL_PATH_UNLESS(from.dim() == 2);
        P = from.size(1);
    }
    GENERAL_PATH_UNLESS(P > 0 && D.is(F32, {H}) && u.is(F32, {Bt, H}) && x_prev.is(C64, {Bt, P}, true) && first.is(U8, {Bt}, true));
    at::Tensor x = xo.t ? *xo.t : empty({Bt, P}, C64, *u.t), y = yo.t ? *yo.t : empty({Bt, H}, F32, *u.t);
    CALL(ssm_step, plan.t->data_ptr(), (size_t)plan.t->numel(), D.f32(), u.f32(), x_prev.c64(), first.u8(), Bt, H, P, c64(x), f32(y), s);
    return tuple({&x, &y});
    TRY_END
}

// (plan, D, dy, dx, is_first, P, want_dx_prev, stream)
ENTRY(step_bwd)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 8 && PyLong_Check(a[5]));
    Arg plan(a[0]), D(a[1]), dy(a[2]), dx(a[3]), first(a[4]);
    void *s;
    GENERAL_PATH_UNLESS(plan.t && dy.dim() == 2 && stream_of(a[7], nullptr, s));
    const int64_t Bt = dy.size(0), H = dy.size(1), P = PyLong_AsLongLong(a[5]);
    if (PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
    GENERAL_PATH_UNLESS(P > 0 && D.is(F32, {H}) && dy.is(F32, {Bt, H}) && dx.is(C64, {Bt, P}, true) && first.is(U8, {Bt}, true));
    at::Tensor gx = empty({Bt, P}, C64, *dy.t), du = empty({Bt, H}, F32, *dy.t), dp;
    if (yes(a[6])) dp = empty({Bt, P}, C64, *dy.t);
    CALL(ssm_step_bwd, plan.t->data_ptr(), (size_t)plan.t->numel(), D.f32(), dy.f32(), dx.c64(), first.u8(), Bt, H, P, c64(gx), f32(du),
                      c64(dp), s);
    return tuple({&gx, &du, &dp});
    TRY_END
}

bool two_floats(PyObject *p, PyObject *q, float &x, float &y)
{
    const double dx = PyFloat_AsDouble(p), dy = PyFloat_AsDouble(q);
    if (PyErr_Occurred()) { PyErr_Clear(); return false; }
    x = (float)dx; y = (float)dy;
    return true;
}

// (reward, cont, value, gamma, lambda, ret, stream)
ENTRY(lambda_return)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 7);
    Arg r(a[0]), c(a[1]), v(a[2]), o(a[5]);
    void *s;
    float gamma, lam;
    GENERAL_PATH_UNLESS(r.dim() == 2 && stream_of(a[6], nullptr, s) && two_floats(a[3], a[4], gamma, lam));
    const int64_t T = r.size(0), N = r.size(1);
    GENERAL_PATH_UNLESS(r.is(F32, {T, N}) && c.is(F32, {T, N}) && v.is(F32, {T, N}) && o.is(F32, {T, N}, true));
    at::Tensor ret = o.t ? *o.t : empty({T, N}, F32, *r.t);
    CALL(ssm_lambda_return, r.f32(), c.f32(), v.f32(), gamma, lam, T, N, f32(ret), s);
    return wrap(ret);
    TRY_END
}

// (cont, value, ret, dret, gamma, lambda, stream)
ENTRY(lambda_return_bwd)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 7);
    Arg c(a[0]), v(a[1]), r(a[2]), d(a[3]);
    void *s;
    float gamma, lam;
    GENERAL_PATH_UNLESS(c.dim() == 2 && stream_of(a[6], nullptr, s) && two_floats(a[4], a[5], gamma, lam));
    const int64_t T = c.size(0), N = c.size(1);
    GENERAL_PATH_UNLESS(c.is(F32, {T, N}) && v.is(F32, {T, N}) && r.is(F32, {T, N}) && d.is(F32, {T, N}));
    at::Tensor dr = empty({T, N}, F32, *c.t), dc = empty({T, N}, F32, *c.t), dv = empty({T, N}, F32, *c.t);
    CALL(ssm_lambda_return_bwd, c.f32(), v.f32(), r.f32(), d.f32(), gamma, lam, T, N, f32(dr), f32(dc), f32(dv), s);
    return tuple({&dr, &dc, &dv});
    TRY_END
}

// (A_bar, v, is_first, x0, want_x_last, workspace, stream) -> x_last or None, as a tuple of one
ENTRY(scan_states)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 7);
    Arg A(a[0]), v(a[1]), first(a[2]), x0(a[3]), ws(a[5]);
    void *s;
    GENERAL_PATH_UNLESS(v.dim() == 3 && stream_of(a[6], &ws, s));
    const int64_t Bt = v.size(0), L = v.size(1), P = v.size(2);
    GENERAL_PATH_UNLESS(A.is(C64, {P}) && v.is(C64, {Bt, L, P}) && first.is(U8, {Bt, L}, true) && x0.is(C64, {Bt, P}, true));
    Workspace w(ws, ws.none ? ssm_workspace_bytes(Bt, L, 1, P, 0) : 0, *v.t);
    GENERAL_PATH_UNLESS(!w.bad);
    at::Tensor xl;
    if (yes(a[4])) xl = empty({Bt, P}, C64, *v.t);
    CALL(ssm_scan_states, A.c64(), v.ptr<ssm_c64>(), first.u8(), x0.c64(), Bt, L, P, c64(xl), w.p, w.n, s);
    return tuple({&xl});
    TRY_END
}

// (A_bar, gx, x, is_first, x0, want_dx0, workspace, stream) -> (dA_bar, dx0 or None)
ENTRY(scan_states_reverse)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 8);
    Arg A(a[0]), g(a[1]), x(a[2]), first(a[3]), x0(a[4]), ws(a[6]);
    void *s;
    GENERAL_PATH_UNLESS(g.dim() == 3 && stream_of(a[7], &ws, s));
    const int64_t Bt = g.size(0), L = g.size(1), P = g.size(2);
    GENERAL_PATH_UNLESS(A.is(C64, {P}) && g.is(C64, {Bt, L, P}) && x.is(C64, {Bt, L, P}) && first.is(U8, {Bt, L}, true) &&
                        x0.is(C64, {Bt, P}, true));
    Workspace w(ws, ws.none ? ssm_workspace_bytes(Bt, L, 1, P, 1) : 0, *g.t);
    GENERAL_PATH_UNLESS(!w.bad);
    at::Tensor dA = empty({P}, C64, *g.t), dx0;
    if (yes(a[5])) dx0 = empty({Bt, P}, C64, *g.t);
    CALL(ssm_scan_states_reverse, A.c64(), g.ptr<ssm_c64>(), x.c64(), first.u8(), x0.c64(), Bt, L, P, c64(dA), c64(dx0), w.p, w.n, s);
    return tuple({&dA, &dx0});
    TRY_END
}

// (u, W, want_gate, workspace, y, gate, stream)
ENTRY(half_glu_fwd)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 7);
    Arg u(a[0]), W(a[1]), ws(a[3]), yo(a[4]), go(a[5]);
    void *s;
    GENERAL_PATH_UNLESS(u.dim() == 2 && stream_of(a[6], &ws, s));
    const int64_t T = u.size(0), H = u.size(1);
    GENERAL_PATH_UNLESS(u.is(F32, {T, H}) && W.is(F32, {H, H}) && yo.is(F32, {T, H}, true) && go.is(F32, {T, H}, true));
    Workspace w(ws, ws.none ? ssm_half_glu_workspace_bytes(T, H, 0) : 0, *u.t);
    GENERAL_PATH_UNLESS(!w.bad);
    at::Tensor y = yo.t ? *yo.t : empty({T, H}, F32, *u.t), gate;
    if (go.t) gate = *go.t;
    else if (yes(a[2])) gate = empty({T, H}, F32, *u.t);
    CALL(ssm_half_glu_fwd, u.f32(), W.f32(), T, H, f32(y), f32(gate), w.p, w.n, s);
    return tuple({&y, &gate});
    TRY_END
}

// (u, W, gate, dy, workspace, du, dW, stream)
ENTRY(half_glu_bwd)
{
    TRY_BEGIN
    GENERAL_PATH_UNLESS(n == 8);
    Arg u(a[0]), W(a[1]), g(a[2]), dy(a[3]), ws(a[4]), duo(a[5]), dWo(a[6]);
    void *s;
    GENERAL_PATH_UNLESS(u.dim() == 2 && stream_of(a[7], &ws, s));
    const int64_t T = u.size(0), H = u.size(1);
    GENERAL_PATH_UNLESS(u.is(F32, {T, H}) && W.is(F32, {H, H}) && g.is(F32, {T, H}) && dy.is(F32, {T, H}) && duo.is(F32, {T, H}, true) &&
                        dWo.is(F32, {H, H}, true));
    Workspace w(ws, ws.none ? ssm_half_glu_workspace_bytes(T, H, 1) : 0, *u.t);
    GENERAL_PATH_UNLESS(!w.bad);
    at::Tensor du = duo.t ? *duo.t : empty({T, H}, F32, *u.t), dW = dWo.t ? *dWo.t : empty({H, H}, F32, *u.t);
    CALL(ssm_half_glu_bwd, u.f32(), W.f32(), g.f32(), dy.f32(), T, H, f32(du), f32(dW), w.p, w.n, s);
    return tuple({&du, &dW});
    TRY_END
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(scan_fwd), METHOD(scan_bwd), METHOD(block_fwd), METHOD(block_bwd), METHOD(step_prepare), METHOD(step),
                         METHOD(step_bwd), METHOD(lambda_return), METHOD(lambda_return_bwd), METHOD(scan_states),
                         METHOD(scan_states_reverse), METHOD(half_glu_fwd), METHOD(half_glu_bwd), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ssmbind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__ssmbind(void) { return PyModule_Create(&module); }
