// The tensor entry points of the Python package (sdpa, sdpa_kv, sdpa_paged, sdpa_backward) in native code: argument
// checks, output and workspace tensors from torch's allocator, the current stream, and one call into the C-ABI of
// include/tiled_sdpa.h.
//
// Why native: a short call is bound by the host.  One forward call of a small problem (B=1 H=2 S=128 D=64, a kernel of
// 4.4 us) took 8.7 us of host time through Python attribute reads, data_ptr() calls and ctypes argument conversion, a
// decoding step with splits (two kernels, a workspace query, two allocations) 17.5 us, a backward call 22-28 us.  The
// same calls take 5.1, 8.6 and 12-17 us here; most of what is left is the launches.
//
// Each function takes every argument of its Python wrapper by position and returns the result object, or the status
// code (a Python int) of a call that the library refused; the wrapper turns that into TiledSdpaError.
#include <Python.h>

#include <cmath>
#include <limits>

#include <ATen/core/Tensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "tiled_sdpa.h"

namespace {

// thrown with a Python error set
struct PyFail {};

[[noreturn]] void fail(const char *text)
{
    PyErr_SetString(PyExc_ValueError, text);
    throw PyFail{};
}

[[noreturn]] void fail_named(const char *name, const char *text)
{
    PyErr_Format(PyExc_ValueError, "%s %s", name, text);
    throw PyFail{};
}

// Tensor arguments are borrowed from the caller's references; THPVariable_Unpack only looks inside.
const at::Tensor &device_tensor(PyObject *obj, const char *name)
{
    if (!THPVariable_Check(obj)) fail_named(name, "must be a device tensor");
    const at::Tensor &t = THPVariable_Unpack(obj);
    if (!t.is_cuda()) fail_named(name, "must be a device tensor");
    return t;
}

const at::Tensor &heads_tensor(PyObject *obj, const char *name)
{
    const at::Tensor &t = device_tensor(obj, name);
    if (t.dim() != 4 || !t.is_contiguous()) fail_named(name, "must be contiguous [B, H, S, D]");
    return t;
}

int element_type(const at::Tensor &t)
{
    if (t.scalar_type() == at::kHalf) return TSDPA_F16;
    if (t.scalar_type() == at::kBFloat16) return TSDPA_BF16;
    fail("dtype must be float16 or bfloat16");
}

void same_type(const at::Tensor &q, const at::Tensor &k, const at::Tensor &v)
{
    if ((q.scalar_type() != at::kHalf && q.scalar_type() != at::kBFloat16) || k.scalar_type() != q.scalar_type() ||
        v.scalar_type() != q.scalar_type())
        fail("q, k, v must share dtype float16 or bfloat16");
}

int as_int(PyObject *obj)
{
    const long x = PyLong_AsLong(obj);
    if (x == -1 && PyErr_Occurred()) throw PyFail{};
    if (x < std::numeric_limits<int>::min() || x > std::numeric_limits<int>::max()) {
        PyErr_SetString(PyExc_OverflowError, "argument does not fit a 32-bit integer");
        throw PyFail{};
    }
    return (int)x;
}

bool as_bool(PyObject *obj)
{
    const int x = PyObject_IsTrue(obj);
    if (x < 0) throw PyFail{};
    return x != 0;
}

unsigned as_flags(PyObject *flags, PyObject *causal)
{
    const unsigned long x = PyLong_AsUnsignedLongMask(flags);
    if (x == (unsigned long)-1 && PyErr_Occurred()) throw PyFail{};
    return (unsigned)x | (as_bool(causal) ? (unsigned)TSDPA_FLAG_CAUSAL : 0u);
}

float as_scale(PyObject *obj)
{
    if (obj == Py_None) return std::numeric_limits<float>::quiet_NaN();
    const double x = PyFloat_AsDouble(obj);
    if (x == -1.0 && PyErr_Occurred()) throw PyFail{};
    return (float)x;
}

struct Tile { int m = 0, n = 0; };

Tile as_tile(PyObject *obj)
{
    Tile t;
    if (obj == Py_None) return t;
    PyObject *seq = PySequence_Fast(obj, "tile must be (tile_m, tile_n)");
    if (!seq) throw PyFail{};
    if (PySequence_Fast_GET_SIZE(seq) != 2) {
        Py_DECREF(seq);
        fail("tile must be (tile_m, tile_n)");
    }
    PyObject *const *items = PySequence_Fast_ITEMS(seq);
    try {
        t.m = as_int(items[0]);
        t.n = as_int(items[1]);
    } catch (...) {
        Py_DECREF(seq);
        throw;
    }
    Py_DECREF(seq);
    return t;
}

// Lets other Python threads run while the allocator or the launch may block (a full queue, say, that waits for a host function
// of another thread).
struct NoGil {
    PyThreadState *state = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(state); }
};

at::Tensor empty(at::IntArrayRef size, at::ScalarType type, const at::Tensor &like)
{
    const NoGil without;
    return at::Tensor(at::detail::empty_cuda(size, type, like.device(), std::nullopt));
}

// Makes the tensors' device current for the call if it is not, and names the stream that is current on it.
struct Launch {
    c10::OptionalDeviceGuard guard;
    void *stream;
    explicit Launch(const at::Tensor &q)
    {
        const c10::DeviceIndex index = q.device().index();
        if (c10::hip::current_device() != index) guard.reset_device(q.device());
        stream = (void *)c10::hip::getCurrentHIPStream(index).stream();
    }
};

// (the arguments are evaluated before the lock is let go)
template <typename... P, typename... A> int without_gil(int (*call)(P...), A... args)
{
    const NoGil without;
    return call(args...);
}

void *data(const at::Tensor &t) { return t.data_ptr(); }

bool same_sizes(const at::Tensor &a, const at::Tensor &b) { return a.sizes() == b.sizes(); }

// `out` of the caller, checked against `like`, or a new tensor of that shape
at::Tensor output(PyObject *obj, const at::Tensor &like, const char *complaint)
{
    if (obj == Py_None) return empty(like.sizes(), like.scalar_type(), like);
    if (!THPVariable_Check(obj)) fail(complaint);
    const at::Tensor &t = THPVariable_Unpack(obj);
    if (!same_sizes(t, like) || t.scalar_type() != like.scalar_type() || !t.is_contiguous() || t.device() != like.device())
        fail(complaint);
    return t;
}

// The object to hand back for a tensor: the caller's own if they passed one.
PyObject *give(PyObject *passed, const at::Tensor &t)
{
    if (passed != Py_None) {
        Py_INCREF(passed);
        return passed;
    }
    return THPVariable_Wrap(t);
}

PyObject *result(int status, PyObject *out_obj, const at::Tensor &out, bool with_lse, PyObject *lse_obj, const at::Tensor &lse)
{
    if (status != TSDPA_OK) return PyLong_FromLong(status);
    PyObject *o = give(out_obj, out);
    if (!o || !with_lse) return o;
    PyObject *l = give(lse_obj, lse);
    if (!l) {
        Py_DECREF(o);
        return nullptr;
    }
    PyObject *pair = PyTuple_New(2);
    if (!pair) {
        Py_DECREF(o);
        Py_DECREF(l);
        return nullptr;
    }
    PyTuple_SET_ITEM(pair, 0, o);
    PyTuple_SET_ITEM(pair, 1, l);
    return pair;
}

struct Workspace {
    at::Tensor held;
    void *ptr = nullptr;
    unsigned long long bytes = 0;
    Workspace() = default;
    // the caller's buffer, or `need` bytes of torch's.  The kernels write to it as to one range of bytes: it has to be that,
    // and on the device of the call (of a call that needs none it is not looked at)
    Workspace(PyObject *obj, unsigned long long need, const at::Tensor &like)
    {
        if (obj != Py_None) {
            if (!THPVariable_Check(obj)) fail("workspace must be a device tensor");
            held = THPVariable_Unpack(obj);
            if (need > 0 && (held.device() != like.device() || !held.is_non_overlapping_and_dense()))
                fail("workspace must be a dense tensor on the device of q");
        } else if (need > 0) {
            held = empty({(int64_t)need}, at::kByte, like);
        } else {
            return;
        }
        ptr = data(held);
        bytes = (unsigned long long)held.numel() * held.element_size();
    }
};

void need_args(Py_ssize_t got, Py_ssize_t want)
{
    if (got == want) return;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, got);
    throw PyFail{};
}

// Runs a function body; C++ exceptions (torch's allocator out of memory among them) become Python's.
template <typename F> PyObject *guarded(F &&body)
{
    try {
        return body();
    } catch (const PyFail &) {
        return nullptr;
    } catch (...) {
        return torch::translate_exception_to_python(std::current_exception()), nullptr;
    }
}

// sdpa(q, k, v, causal, scale, return_lse, out, lse_out, tile, flags)
PyObject *call_sdpa(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        need_args(n, 10);
        const at::Tensor &q = heads_tensor(args[0], "q"), &k = heads_tensor(args[1], "k"), &v = heads_tensor(args[2], "v");
        const unsigned flags = as_flags(args[9], args[3]);
        const float scale = as_scale(args[4]);
        const bool with_lse = as_bool(args[5]);
        const Tile tile = as_tile(args[8]);
        same_type(q, k, v);
        if (!same_sizes(q, k) || !same_sizes(q, v) || k.device() != q.device() || v.device() != q.device())
            fail("q, k, v must have identical shape and device");
        const at::IntArrayRef s = q.sizes();
        at::Tensor out = output(args[6], q, "out must match q in shape, dtype, device and be contiguous");
        at::Tensor lse;
        if (with_lse) {
            if (args[7] != Py_None) {
                static const char text[] = "lse_out must be contiguous float32 [B, H, S] on the device of q";
                if (!THPVariable_Check(args[7])) fail(text);
                lse = THPVariable_Unpack(args[7]);
                if (lse.sizes() != s.slice(0, 3) || lse.scalar_type() != at::kFloat || !lse.is_contiguous() || lse.device() != q.device())
                    fail(text);
            } else {
                lse = empty(s.slice(0, 3), at::kFloat, q);
            }
        }
        const Launch on(q);
        const int st = without_gil(tiled_sdpa_fwd_ex, data(q), data(k), data(v), data(out), with_lse ? (float *)data(lse) : nullptr,
                                         (int)s[0], (int)s[1], (int)s[2], (int)s[3], scale, element_type(q), on.stream,
                                         tile.m, tile.n, flags);
        return result(st, args[6], out, with_lse, args[7], lse);
    });
}

// The split count of a call that leaves it to the library (which sees B * Hkv heads of G * Sq rows each).  A tile that the library
// does not offer is for the call itself to refuse, after the checks that come before that one.
int heuristic_splits(int B, int H, int Hkv, int Sq, int Skv, int D, int dtype, unsigned flags, bool drop_causal, Tile tile, int *splits)
{
    const int st = tiled_sdpa_kv_tile_splits(B, Hkv, (int)((int64_t)(H / Hkv) * Sq), Skv, D, dtype,
                                             drop_causal ? flags & ~(unsigned)TSDPA_FLAG_CAUSAL : flags, tile.m, tile.n, splits);
    return st == TSDPA_ERR_BAD_TILE ? TSDPA_OK : st;
}

// sdpa_kv(q, k, v, causal, scale, splits, return_lse, out, workspace, tile, flags, kv_lens)
PyObject *call_sdpa_kv(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        need_args(n, 12);
        const at::Tensor &q = heads_tensor(args[0], "q"), &k = heads_tensor(args[1], "k"), &v = heads_tensor(args[2], "v");
        const unsigned flags = as_flags(args[10], args[3]);
        const float scale = as_scale(args[4]);
        int splits = args[5] == Py_None ? 0 : as_int(args[5]);
        const bool with_lse = as_bool(args[6]);
        const Tile tile = as_tile(args[9]);
        same_type(q, k, v);
        const at::IntArrayRef s = q.sizes(), t = k.sizes();
        if (!same_sizes(k, v) || s[0] != t[0] || s[3] != t[3]) fail("q must be [B, H, Sq, D] and k, v [B, Hkv, Skv, D]");
        if (t[1] == 0 || s[1] % t[1] != 0) fail("the number of query heads must be a multiple of the number of key/value heads");
        if (k.device() != q.device() || v.device() != q.device()) fail("q, k, v must be on one device");
        const int *lens = nullptr;
        if (args[11] != Py_None) {
            static const char text[] = "kv_lens must be a contiguous int32 tensor [B] on the device of q";
            if (!THPVariable_Check(args[11])) fail(text);
            const at::Tensor &l = THPVariable_Unpack(args[11]);
            if (l.scalar_type() != at::kInt || l.device() != q.device() || l.dim() != 1 || l.size(0) != s[0] || !l.is_contiguous())
                fail(text);
            lens = (const int *)data(l);
        }
        const int B = (int)s[0], H = (int)s[1], Sq = (int)s[2], D = (int)s[3], Hkv = (int)t[1], Skv = (int)t[2];
        const int dtype = element_type(q);
        at::Tensor out = output(args[7], q, "out must match q in shape, dtype, device and be contiguous"), lse;
        if (with_lse) lse = empty(s.slice(0, 3), at::kFloat, q);
        const bool heuristic = splits == 0;
        if (heuristic) {
            const int st = heuristic_splits(B, H, Hkv, Sq, Skv, D, dtype, flags, H != Hkv, tile, &splits);
            if (st != TSDPA_OK) return PyLong_FromLong(st);
        }
        const Workspace ws(args[8], tiled_sdpa_kv_workspace_bytes(B, H, Sq, D, splits), q);
        if (heuristic && args[8] != Py_None) splits = 0;      // (what fits the caller's buffer: the library decides)
        const Launch on(q);
        const int st = without_gil(tiled_sdpa_fwd_kvcache, data(q), data(k), data(v), data(out), with_lse ? (float *)data(lse) : nullptr, lens,
                                              B, H, Hkv, Sq, Skv, D, scale, dtype, on.stream, tile.m, tile.n, flags, splits,
                                              ws.ptr, ws.bytes);
        return result(st, args[7], out, with_lse, Py_None, lse);
    });
}

// sdpa_paged(q, k_pages, v_pages, kv_lens, block_table, causal, scale, splits, return_lse, out, workspace, tile, flags)
PyObject *call_sdpa_paged(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        need_args(n, 13);
        const at::Tensor *tensors[3];
        static const char *names[3] = {"q", "k_pages", "v_pages"};
        for (int i = 0; i < 3; ++i) {
            if (!THPVariable_Check(args[i])) fail_named(names[i], "must be a contiguous 4-d device tensor");
            tensors[i] = &THPVariable_Unpack(args[i]);
            if (!tensors[i]->is_cuda() || tensors[i]->dim() != 4 || !tensors[i]->is_contiguous())
                fail_named(names[i], "must be a contiguous 4-d device tensor");
        }
        const at::Tensor &q = *tensors[0], &k = *tensors[1], &v = *tensors[2];
        const unsigned flags = as_flags(args[12], args[5]);
        const float scale = as_scale(args[6]);
        int splits = args[7] == Py_None ? 0 : as_int(args[7]);
        const bool with_lse = as_bool(args[8]);
        const Tile tile = as_tile(args[11]);
        if ((q.scalar_type() != at::kHalf && q.scalar_type() != at::kBFloat16) || k.scalar_type() != q.scalar_type() ||
            v.scalar_type() != q.scalar_type())
            fail("q, k_pages, v_pages must share dtype float16 or bfloat16");
        const at::IntArrayRef s = q.sizes(), t = k.sizes();
        if (!same_sizes(k, v) || t[3] != s[3] || k.device() != q.device() || v.device() != q.device())
            fail("k_pages, v_pages must be [P, Hkv, block_rows, D] on the device of q");
        if (t[1] == 0 || s[1] % t[1] != 0) fail("the number of query heads must be a multiple of the number of key/value heads");
        if (!THPVariable_Check(args[3])) fail("kv_lens must be a contiguous int32 device tensor");
        if (!THPVariable_Check(args[4])) fail("block_table must be a contiguous int32 device tensor");
        const at::Tensor &lens = THPVariable_Unpack(args[3]), &table = THPVariable_Unpack(args[4]);
        if (lens.scalar_type() != at::kInt || lens.device() != q.device() || !lens.is_contiguous() || lens.dim() != 1 || lens.size(0) != s[0])
            fail("kv_lens must be a contiguous int32 device tensor");
        if (table.scalar_type() != at::kInt || table.device() != q.device() || !table.is_contiguous())
            fail("block_table must be a contiguous int32 device tensor");
        if (table.dim() != 2 || table.size(0) != s[0]) fail("block_table must be [B, max_blocks]");
        const int B = (int)s[0], H = (int)s[1], Sq = (int)s[2], D = (int)s[3], Hkv = (int)t[1], block_rows = (int)t[2];
        const int max_blocks = (int)table.size(1), dtype = element_type(q);
        at::Tensor out = output(args[9], q, "out must match q in shape, dtype, device and be contiguous"), lse;
        if (with_lse) lse = empty(s.slice(0, 3), at::kFloat, q);
        const bool heuristic = splits == 0;
        if (heuristic) {
            const int64_t rows = (int64_t)max_blocks * block_rows;
            if (rows > std::numeric_limits<int>::max()) return PyLong_FromLong(TSDPA_ERR_BAD_SHAPE);
            const int st = heuristic_splits(B, H, Hkv, Sq, rows > 1 ? (int)rows : 1, D, dtype, flags, true, tile, &splits);
            if (st != TSDPA_OK) return PyLong_FromLong(st);
        }
        const Workspace ws(args[10], tiled_sdpa_kv_workspace_bytes(B, H, Sq, D, splits), q);
        if (heuristic && args[10] != Py_None) splits = 0;
        const Launch on(q);
        const int st = without_gil(tiled_sdpa_fwd_paged, data(q), data(k), data(v), data(out), with_lse ? (float *)data(lse) : nullptr,
                                            (const int *)data(lens), (const int *)data(table), B, H, Hkv, Sq, max_blocks,
                                            block_rows, D, scale, dtype, on.stream, tile.m, tile.n, flags, splits, ws.ptr, ws.bytes);
        return result(st, args[9], out, with_lse, Py_None, lse);
    });
}

// sdpa_backward(q, k, v, o, dout, lse, causal, scale, workspace, grads)
PyObject *call_sdpa_backward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded([&]() -> PyObject * {
        need_args(n, 10);
        const at::Tensor &q = heads_tensor(args[0], "q"), &k = heads_tensor(args[1], "k"), &v = heads_tensor(args[2], "v");
        const at::Tensor &o = heads_tensor(args[3], "o"), &dout = heads_tensor(args[4], "dout");
        auto agree = [&](const at::Tensor &t, const at::Tensor &like) {
            if (!same_sizes(t, like) || t.scalar_type() != q.scalar_type() || t.device() != q.device())
                fail("q, o, dout and k, v must agree in shape, dtype and device");
        };
        agree(k, k);
        agree(v, k);
        agree(o, q);
        agree(dout, q);
        const int dtype = element_type(q);
        const at::IntArrayRef s = q.sizes(), t = k.sizes();
        if (t[0] != s[0] || t[2] != s[2] || t[3] != s[3] || t[1] == 0 || s[1] % t[1] != 0)
            fail("k, v must be [B, Hkv, S, D] with H a multiple of Hkv");
        if (!THPVariable_Check(args[5])) fail("lse must be contiguous float32 [B, H, S] on the same device");
        const at::Tensor &lse = THPVariable_Unpack(args[5]);
        if (lse.sizes() != s.slice(0, 3) || lse.scalar_type() != at::kFloat || !lse.is_contiguous() || lse.device() != q.device())
            fail("lse must be contiguous float32 [B, H, S] on the same device");
        const unsigned flags = as_bool(args[6]) ? (unsigned)TSDPA_FLAG_CAUSAL : 0u;
        const float scale = as_scale(args[7]);
        at::Tensor grad[3];
        if (args[9] == Py_None) {
            grad[0] = empty(s, q.scalar_type(), q);
            grad[1] = empty(t, q.scalar_type(), q);
            grad[2] = empty(t, q.scalar_type(), q);
        } else {
            static const char *complaints[3] = {"dq must match q in shape, dtype, device and be contiguous",
                                                "dk must match k in shape, dtype, device and be contiguous",
                                                "dv must match k in shape, dtype, device and be contiguous"};
            PyObject *seq = PySequence_Fast(args[9], "grads must be (dq, dk, dv)");
            if (!seq) throw PyFail{};
            if (PySequence_Fast_GET_SIZE(seq) < 3) {
                Py_DECREF(seq);
                fail("grads must be (dq, dk, dv)");
            }
            try {
                for (int i = 0; i < 3; ++i) {
                    PyObject *item = PySequence_Fast_GET_ITEM(seq, i);
                    if (item == Py_None) fail(complaints[i]);
                    grad[i] = output(item, i == 0 ? q : k, complaints[i]);
                }
            } catch (...) {
                Py_DECREF(seq);
                throw;
            }
            Py_DECREF(seq);
        }
        const int B = (int)s[0], H = (int)s[1], S = (int)s[2], D = (int)s[3];
        const unsigned long long least = tiled_sdpa_bwd_workspace_bytes(B, H, S);
        Workspace ws;
        if (args[8] == Py_None) {
            // Without memory for the sums of dQ the call takes the passes that need none, as it did before there were such sums.  (Whatever the
            // allocator's error: without its cache it reports HIP's own.  One that is not about the size comes again.)
            const unsigned long long full = tiled_sdpa_bwd_full_workspace_bytes(B, H, (int)t[1], S, D, flags);
            try {
                ws = Workspace(args[8], full, q);
            } catch (const c10::Error &) {
                if (full == least) throw;
            }
        }
        if (!ws.ptr) ws = Workspace(args[8], least, q);
        const Launch on(q);
        const int st = without_gil(tiled_sdpa_bwd_gqa, data(q), data(k), data(v), data(o), data(dout), (const float *)data(lse), data(grad[0]),
                                          data(grad[1]), data(grad[2]), B, H, (int)t[1], S, D, scale, dtype, flags, ws.ptr,
                                          ws.bytes, on.stream);
        if (st != TSDPA_OK) return PyLong_FromLong(st);
        if (args[9] != Py_None) {
            Py_INCREF(args[9]);
            return args[9];
        }
        PyObject *all = PyTuple_New(3);
        if (!all) return nullptr;
        for (int i = 0; i < 3; ++i) {
            PyObject *g = THPVariable_Wrap(grad[i]);
            if (!g) {
                Py_DECREF(all);
                return nullptr;
            }
            PyTuple_SET_ITEM(all, i, g);
        }
        return all;
    });
}

PyMethodDef methods[] = {
    {"sdpa", (PyCFunction)(void (*)(void))call_sdpa, METH_FASTCALL, nullptr},
    {"sdpa_kv", (PyCFunction)(void (*)(void))call_sdpa_kv, METH_FASTCALL, nullptr},
    {"sdpa_paged", (PyCFunction)(void (*)(void))call_sdpa_paged, METH_FASTCALL, nullptr},
    {"sdpa_backward", (PyCFunction)(void (*)(void))call_sdpa_backward, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_calls", "tensor entry points of tiled SDPA", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_calls(void) { return PyModule_Create(&module); }
