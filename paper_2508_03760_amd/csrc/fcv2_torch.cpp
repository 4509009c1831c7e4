// fcv2_torch.cpp -- CPython binding of libfcv2 for torch tensors: the marshalling of every call of fcv2.py in native code.
//
// A codec call on a decode-sized payload keeps the GPU busy for 2 to 7 us; reading shapes, pointers and the stream through
// Python and ctypes took 10 us a call (15 with eight peers, 18 for a dispatch) and was what such a call cost.  Here the
// tensors are read through the C++ interface of torch and the whole call, argument checks included, is about 3 us, most of
// it the runtime's own launch.  Nothing is kept between calls, and the interpreter lock is released around the launch.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>

#include "../../include/fcv2.h"
#include "fcv2_fresh.h"

namespace {

PyObject* g_error = nullptr;          // Fcv2Error
PyObject* g_out_of_memory = nullptr;  // torch.OutOfMemoryError

struct Raised {};  // a Python exception is set

[[noreturn]] void fail(const char* msg) {
    PyErr_SetString(g_error, msg);
    throw Raised{};
}
void check(int rc, const char* what) {
    if (rc == FCV2_OK) return;
    PyErr_Format(g_error, "%s: %s (%d)", what, fcv2_status_string(rc), rc);
    throw Raised{};
}

uint64_t as_u64(PyObject* o) {
    uint64_t v;
    if (PyLong_Check(o)) {
        v = PyLong_AsUnsignedLongLongMask(o);
    } else {
        PyObject* i = PyNumber_Index(o);
        if (!i) throw Raised{};
        v = PyLong_AsUnsignedLongLongMask(i);
        Py_DECREF(i);
    }
    if (v == (uint64_t)-1 && PyErr_Occurred()) throw Raised{};
    return v;
}
uint32_t as_u32(PyObject* o) { return (uint32_t)as_u64(o); }

const at::Tensor& tensor(PyObject* o, const char* what) {
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a torch.Tensor, not %s", what, Py_TYPE(o)->tp_name);
        throw Raised{};
    }
    return THPVariable_Unpack(o);
}
void* dev(const at::Tensor& t, const char* what) {
    if (!t.is_cuda() || !t.is_contiguous()) {
        PyErr_Format(g_error, "%s must be a contiguous device tensor", what);
        throw Raised{};
    }
    return t.data_ptr();
}
at::ScalarType dtype(PyObject* o) {
    if (!THPDtype_Check(o)) {
        PyErr_SetString(PyExc_TypeError, "out_dtype must be a torch.dtype");
        throw Raised{};
    }
    return reinterpret_cast<THPDtype*>(o)->scalar_type;
}
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

fcv2_fmt_t fmt_of(PyObject* bits, PyObject* group, PyObject* flags) { return {as_u32(bits), as_u32(group), as_u32(flags)}; }
fcv2_fmt_t fmt_of(PyObject* triple) {
    PyObject* f = PySequence_Fast(triple, "a format is (bits, group, flags)");
    if (!f) throw Raised{};
    fcv2_fmt_t r{};
    const bool three = PySequence_Fast_GET_SIZE(f) == 3;
    if (three) {
        PyObject** it = PySequence_Fast_ITEMS(f);
        try {
            r = fmt_of(it[0], it[1], it[2]);
        } catch (...) {
            Py_DECREF(f);
            throw;
        }
    }
    Py_DECREF(f);
    if (!three) {
        PyErr_SetString(PyExc_TypeError, "a format is (bits, group, flags)");
        throw Raised{};
    }
    return r;
}
fcv2_layout_t layout(uint64_t n, const fcv2_fmt_t& f, uint32_t align) {
    fcv2_layout_t l;
    check(fcv2_get_layout(n, &f, align, &l), "fcv2_get_layout");
    return l;
}

// Up to FCV2_MAX_PEERS records of a Python sequence: every one a uint8 tensor of at least `bytes`.
struct Records {
    PyObject* seq;
    int n;
    explicit Records(PyObject* o) : seq(PySequence_Fast(o, "the records must be a sequence of tensors")) {
        if (!seq) throw Raised{};
        const Py_ssize_t k = PySequence_Fast_GET_SIZE(seq);
        n = k > 1 << 20 ? 1 << 20 : (int)k;
    }
    Records(const Records&) = delete;
    ~Records() { Py_DECREF(seq); }
    const at::Tensor& at(int i, const char* what) const { return tensor(PySequence_Fast_GET_ITEM(seq, i), what); }
    void check_sizes(uint64_t bytes, const char* what, const char* message) const {
        for (int i = 0; i < n; ++i) {
            const at::Tensor& t = at(i, what);
            if (t.scalar_type() != at::kByte || (uint64_t)t.numel() < bytes) fail(message);
        }
    }
    void pointers(const void** p, const char* what) const {
        for (int i = 0; i < n; ++i) p[i] = dev(at(i, what), what);
    }
};

at::Tensor new_tensor(at::IntArrayRef shape, at::ScalarType t, const at::Tensor& like) {
    return like.is_cuda() ? at::Tensor(at::detail::empty_cuda(shape, t, like.device(), std::nullopt))
                          : at::empty(shape, at::TensorOptions().dtype(t).device(like.device()));
}

// An optional argument that the caller may have passed: the tensor and the object to hand back.
struct Given {
    PyObject* obj;
    at::Tensor made;
    explicit Given(PyObject* o) : obj(o == Py_None ? nullptr : o) {}
    explicit operator bool() const { return obj != nullptr; }
    const at::Tensor& get(const char* what) const { return obj ? tensor(obj, what) : made; }
    PyObject* result() {
        if (!obj) return THPVariable_Wrap(made);
        Py_INCREF(obj);
        return obj;
    }
};

template <class F> int without_gil(F f) {
    int rc;
    Py_BEGIN_ALLOW_THREADS rc = f();
    Py_END_ALLOW_THREADS return rc;
}

// x, bits, group, flags, out
PyObject* quantize_pack(PyObject* const* a) {
    const at::Tensor& x = tensor(a[0], "x");
    if (x.scalar_type() != at::kBFloat16) fail("x must be bfloat16");
    const uint64_t n = (uint64_t)x.numel();
    const fcv2_fmt_t f = fmt_of(a[1], a[2], a[3]);
    const fcv2_layout_t l = layout(n, f, FCV2_TENSOR_ALIGN);
    Given out(a[4]);
    if (!out)
        out.made = new_tensor({(int64_t)l.total_bytes}, at::kByte, x);
    else if ((uint64_t)out.get("out").numel() < l.total_bytes || out.get("out").scalar_type() != at::kByte)
        fail("out must be a uint8 tensor of at least total_bytes");
    const void* xp = dev(x, "x");
    void *op = dev(out.get("out"), "out"), *st = stream();
    const bool fresh = !out;
    check(without_gil([&] { return fresh ? fcv2_quantize_pack_slices_fresh(xp, n, 1, &f, op, st) : fcv2_quantize_pack(xp, n, &f, op, st); }),
          "fcv2_quantize_pack");
    return out.result();
}

// packed, n, bits, group, flags, out_dtype, out
PyObject* unpack_dequant(PyObject* const* a) {
    const at::Tensor& p = tensor(a[0], "packed");
    const uint64_t n = as_u64(a[1]);
    const fcv2_fmt_t f = fmt_of(a[2], a[3], a[4]);
    const fcv2_layout_t l = layout(n, f, FCV2_TENSOR_ALIGN);
    if (p.scalar_type() != at::kByte || (uint64_t)p.numel() < l.total_bytes) fail("packed must be a uint8 tensor of at least total_bytes");
    const at::ScalarType t = dtype(a[5]);
    if (t != at::kFloat && t != at::kBFloat16) fail("out_dtype must be float32 or bfloat16");
    Given out(a[6]);
    if (!out)
        out.made = new_tensor({(int64_t)n}, t, p);
    else if ((uint64_t)out.get("out").numel() != n || out.get("out").scalar_type() != t)
        fail("out has the wrong size or dtype");
    const void* pp = dev(p, "packed");
    void *op = dev(out.get("out"), "out"), *st = stream();
    const int dt = t == at::kFloat ? FCV2_DT_FP32 : FCV2_DT_BF16;
    check(without_gil([&] { return fcv2_unpack_dequant(pp, n, &f, op, dt, st); }), "fcv2_unpack_dequant");
    return out.result();
}

// x, n_slices, bits, group, flags, out
PyObject* quantize_pack_slices(PyObject* const* a) {
    const at::Tensor& x = tensor(a[0], "x");
    if (x.scalar_type() != at::kBFloat16) fail("x must be bfloat16");
    const uint64_t n = (uint64_t)x.numel();
    const int64_t k = (int64_t)as_u64(a[1]);
    if (k < 1 || n % (uint64_t)k) fail("n must be a multiple of n_slices");
    const fcv2_fmt_t f = fmt_of(a[2], a[3], a[4]);
    const fcv2_layout_t l = layout(n / (uint64_t)k, f, FCV2_TENSOR_ALIGN);
    Given out(a[5]);
    if (!out) {
        out.made = new_tensor({k, (int64_t)l.total_bytes}, at::kByte, x);
    } else {
        const at::Tensor& o = out.get("out");
        if (o.scalar_type() != at::kByte || o.dim() != 2 || o.size(0) != k || (uint64_t)o.size(1) < l.total_bytes)
            fail("out must be a uint8 tensor [n_slices, >= total_bytes]");
    }
    const void* xp = dev(x, "x");
    const uint64_t stride = (uint64_t)out.get("out").size(1);
    void *op = dev(out.get("out"), "out"), *st = stream();
    const bool fresh = !out;
    check(without_gil([&] {
              return fresh ? fcv2_quantize_pack_slices_fresh(xp, n, (uint32_t)k, &f, op, st)
                           : fcv2_quantize_pack_slices(xp, n, (uint32_t)k, &f, op, stride, st);
          }),
          "fcv2_quantize_pack_slices");
    return out.result();
}

// records, n, bits, group, flags, out_dtype, out
PyObject* unpack_dequant_slices(PyObject* const* a) {
    const Records recs(a[0]);
    const uint64_t n = as_u64(a[1]);
    if (recs.n < 1 || n % (uint64_t)recs.n) fail("n must be a multiple of the number of records");
    const fcv2_fmt_t f = fmt_of(a[2], a[3], a[4]);
    const fcv2_layout_t l = layout(n / (uint64_t)recs.n, f, FCV2_TENSOR_ALIGN);
    recs.check_sizes(l.total_bytes, "record", "every record must be a uint8 tensor of at least total_bytes");
    const at::ScalarType t = dtype(a[5]);
    Given out(a[6]);
    if (!out) out.made = new_tensor({(int64_t)n}, t, recs.at(0, "record"));
    const void* p[FCV2_MAX_PEERS];
    if (recs.n > FCV2_MAX_PEERS) check(FCV2_ERR_INVALID_ARG, "fcv2_unpack_dequant_slices");
    recs.pointers(p, "record");
    void *op = dev(out.get("out"), "out"), *st = stream();
    const int dt = t == at::kFloat ? FCV2_DT_FP32 : FCV2_DT_BF16;
    check(without_gil([&] { return fcv2_unpack_dequant_slices(p, (uint32_t)recs.n, n, &f, op, dt, st); }), "fcv2_unpack_dequant_slices");
    return out.result();
}

// peers, n, fmt_in, fmt_out, want_sum, out, sum_out
PyObject* reduce_requant(PyObject* const* a) {
    const uint64_t n = as_u64(a[1]);
    const fcv2_fmt_t fin = fmt_of(a[2]);
    const int other = PyObject_IsTrue(a[3]), want = PyObject_IsTrue(a[4]);
    if (other < 0 || want < 0) throw Raised{};
    const fcv2_fmt_t fout = other ? fmt_of(a[3]) : fin;
    const fcv2_layout_t lin = layout(n, fin, FCV2_TENSOR_ALIGN), lout = layout(n, fout, FCV2_TENSOR_ALIGN);
    const Records peers(a[0]);
    if (peers.n < 1 || peers.n > FCV2_MAX_PEERS) fail("1..16 peers");
    peers.check_sizes(lin.total_bytes, "peer", "every peer must be a uint8 tensor of at least total_bytes");
    Given out(a[5]), sum(a[6]);
    if (!out) out.made = new_tensor({(int64_t)lout.total_bytes}, at::kByte, peers.at(0, "peer"));
    if (want && !sum) sum.made = new_tensor({(int64_t)n}, at::kFloat, peers.at(0, "peer"));
    const void* p[FCV2_MAX_PEERS];
    peers.pointers(p, "peer");
    void* op = dev(out.get("out"), "out");
    float* sp = (sum || want) ? (float*)dev(sum.get("sum_out"), "sum_out") : nullptr;
    void* st = stream();
    const auto call = out ? fcv2_reduce_requant : fcv2_reduce_requant_fresh;
    check(without_gil([&] { return call(p, peers.n, n, &fin, &fout, op, sp, st); }), "fcv2_reduce_requant");
    if (!want) return out.result();
    PyObject* pair = PyTuple_New(2);
    if (!pair) throw Raised{};
    PyTuple_SET_ITEM(pair, 0, out.result());
    PyTuple_SET_ITEM(pair, 1, sum.result());
    return pair;
}

// What both dispatch calls read from x, topk_ids, E, bits, group, flags.
struct Routed {
    const at::Tensor &x, &ids;
    uint32_t T, H, K, E;
    fcv2_fmt_t f;
    explicit Routed(PyObject* const* a) : x(tensor(a[0], "x")), ids(tensor(a[1], "topk_ids")) {
        if (x.dim() != 2) {
            PyErr_SetString(PyExc_ValueError, "x must be [T,H]");
            throw Raised{};
        }
        if (ids.dim() < 2) {
            PyErr_SetString(PyExc_IndexError, "topk_ids must be [T,K]");
            throw Raised{};
        }
        T = (uint32_t)x.size(0);
        H = (uint32_t)x.size(1);
        K = (uint32_t)ids.size(1);
        if (x.scalar_type() != at::kBFloat16 || ids.scalar_type() != at::kInt || ids.size(0) != x.size(0))
            fail("x must be [T,H] bfloat16 and topk_ids [T,K] int32");
        E = as_u32(a[2]);
        f = fmt_of(a[3], a[4], a[5]);
    }
};
PyObject* three(Given& a, Given& b, Given& c) {
    PyObject* t = PyTuple_New(3);
    if (!t) throw Raised{};
    PyTuple_SET_ITEM(t, 0, a.result());
    PyTuple_SET_ITEM(t, 1, b.result());
    PyTuple_SET_ITEM(t, 2, c.result());
    return t;
}

// x, topk_ids, E, bits, group, flags, send_buf, expert_offsets, row_src, workspace
PyObject* dispatch_quant(PyObject* const* a) {
    const Routed r(a);
    const fcv2_layout_t l = layout(r.H, r.f, FCV2_ROW_ALIGN);
    const int64_t slots = (int64_t)r.T * r.K;
    Given send(a[6]), offsets(a[7]), src(a[8]), ws(a[9]);
    // The kernels define all of send_buf and row_src only when both are ours; one alone is filled the plain way.
    const bool fresh = !send && !src;
    if (!send) send.made = new_tensor({slots, (int64_t)l.total_bytes}, at::kByte, r.x);
    if (!src) src.made = new_tensor({slots}, at::kInt, r.x);
    if (!send && !fresh) send.made.zero_();
    if (!src && !fresh) src.made.fill_(-1);
    if (!offsets) offsets.made = new_tensor({(int64_t)r.E + 1}, at::kInt, r.x);  // every entry is an output of the call
    size_t need = 0;
    check(fcv2_dispatch_workspace_bytes(r.T, r.K, r.E, &need), "fcv2_dispatch_workspace_bytes");
    if (!ws) ws.made = new_tensor({(int64_t)need}, at::kByte, r.x);
    const void *xp = dev(r.x, "x"), *ip = dev(r.ids, "topk_ids");
    void *sp = dev(send.get("send_buf"), "send_buf"), *ep = dev(offsets.get("expert_offsets"), "expert_offsets"),
         *rp = dev(src.get("row_src"), "row_src"), *wp = dev(ws.get("workspace"), "workspace"), *st = stream();
    const size_t have = (size_t)ws.get("workspace").numel();
    const auto call = fresh ? fcv2_dispatch_quant_fresh : fcv2_dispatch_quant;
    check(without_gil([&] {
              return call(xp, (const int32_t*)ip, r.T, r.H, r.K, r.E, &r.f, sp, (int32_t*)ep, (int32_t*)rp, wp, have, st);
          }),
          "fcv2_dispatch_quant");
    return three(send, offsets, src);
}

// x, topk_ids, E, bits, group, flags, send_buf, expert_offsets, row_src
PyObject* dispatch_quant_noalloc(PyObject* const* a) {
    const Routed r(a);
    const void *xp = dev(r.x, "x"), *ip = dev(r.ids, "topk_ids");
    Given send(a[6]), offsets(a[7]), src(a[8]);
    if (!send || !offsets || !src) {
        PyErr_SetString(PyExc_TypeError, "send_buf, expert_offsets and row_src must be tensors");
        throw Raised{};
    }
    void *sp = dev(send.get("send_buf"), "send_buf"), *ep = dev(offsets.get("expert_offsets"), "expert_offsets"),
         *rp = dev(src.get("row_src"), "row_src"), *st = stream();
    check(without_gil([&] {
              return fcv2_dispatch_quant_noalloc(xp, (const int32_t*)ip, r.T, r.H, r.K, r.E, &r.f, sp, (int32_t*)ep, (int32_t*)rp, st);
          }),
          "fcv2_dispatch_quant_noalloc");
    return three(send, offsets, src);
}

// Every function takes its arguments by position, all of them (fcv2.py fills in the defaults).
template <PyObject* (*F)(PyObject* const*), Py_ssize_t N> PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", N, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Raised&) {
    } catch (const std::exception& e) {  // torch: out of memory and the like
        if (!PyErr_Occurred()) {
            const bool oom = dynamic_cast<const c10::OutOfMemoryError*>(&e) != nullptr;
            PyErr_SetString(oom ? g_out_of_memory : PyExc_RuntimeError, e.what());
        }
    }
    return nullptr;
}

// set_errors(Fcv2Error, torch.OutOfMemoryError)
PyObject* set_errors(PyObject*, PyObject* args) {
    PyObject *error, *out_of_memory;
    if (!PyArg_ParseTuple(args, "OO", &error, &out_of_memory)) return nullptr;
    Py_INCREF(error);
    Py_INCREF(out_of_memory);
    Py_XSETREF(g_error, error);
    Py_XSETREF(g_out_of_memory, out_of_memory);
    Py_RETURN_NONE;
}

#define FCV2_ENTRY(name, n) {#name, (PyCFunction)(void (*)(void))entry<name, n>, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {FCV2_ENTRY(quantize_pack, 5),
                           FCV2_ENTRY(unpack_dequant, 7),
                           FCV2_ENTRY(quantize_pack_slices, 6),
                           FCV2_ENTRY(unpack_dequant_slices, 7),
                           FCV2_ENTRY(reduce_requant, 7),
                           FCV2_ENTRY(dispatch_quant, 10),
                           FCV2_ENTRY(dispatch_quant_noalloc, 9),
                           {"set_errors", set_errors, METH_VARARGS, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fcv2_torch", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fcv2_torch(void) {
    g_error = g_out_of_memory = PyExc_RuntimeError;
    Py_INCREF(g_error);
    Py_INCREF(g_out_of_memory);
    return PyModule_Create(&g_module);
}
