// Native marshalling of the Python binding's calls: tensors in, the C entry point called with their addresses, sizes and the
// current stream.  A call stands in front of kernels of a few microseconds; marshalled in Python through ctypes it cost about
// 6 us of host time, more than the kernel of a decode step takes.
//
// Every function takes plain strided CUDA tensors in the shapes that the entry point wants, outputs included, and returns the
// entry point's status.  Anything else - a subclass, a wrapper of a transform, a missing output, a wrong type or shape -
// returns None and nothing has happened: the binding's Python code then does the call or raises.
#include <Python.h>

#include <string.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include "mx4.h"

namespace {

struct Calls {  // the C entry points, by the addresses that the binding passes in
    decltype(&mx_quantize) quantize;
    decltype(&mx_quantize_mbs) quantize_mbs;
    decltype(&mx_quantize_mbs_pair) quantize_mbs_pair;
    decltype(&mx_quantize_mbs_dynamic) quantize_mbs_dynamic;
    decltype(&mx_quantize_elem) quantize_elem;
    decltype(&mx_dequantize) dequantize;
    decltype(&mx_gemm) gemm;
    decltype(&mx_gemm_mbs) gemm_mbs;
    decltype(&mx_gemm_mbs_grouped) gemm_mbs_grouped;
    decltype(&mx_gemm_mbs_quantize_a) gemm_mbs_quantize_a;
    decltype(&mx_gemm_mbs_elem) gemm_mbs_elem;
    decltype(&mx_gemm_mbs_elem_grouped) gemm_mbs_elem_grouped;
} calls;

struct Declined {};  // the arguments are not what is served here

void need(bool ok) {
    if (!ok) throw Declined();
}

// (the types of the arguments have been looked at: `served`)
const at::Tensor& tensor(PyObject* o) {
    const at::Tensor& t = THPVariable_Unpack(o);
    using K = c10::DispatchKey;
    need(t.defined() && t.is_cuda() && t.layout() == c10::kStrided && t.has_storage() && !t.unsafeGetTensorImpl()->is_python_dispatch() &&
         !t.key_set().has_any(c10::DispatchKeySet({K::Python, K::FuncTorchBatched, K::FuncTorchGradWrapper, K::Functionalize, K::BatchedNestedTensor})));
    return t;
}

template <typename T = uint8_t>
T* address(const at::Tensor& t) {
    return static_cast<T*>(t.data_ptr());
}
// the address of an optional operand array (its shape is not looked at)
const uint8_t* optional(PyObject* o) { return o == Py_None ? nullptr : address(tensor(o)); }

struct Rows {  // a bf16 matrix
    const void* data;
    int64_t rows, K, ld;
};
Rows bf16_rows(PyObject* o) {
    const at::Tensor& t = tensor(o);
    need(t.scalar_type() == at::kBFloat16 && t.dim() == 2);
    const int64_t rows = t.size(0), K = t.size(1), ld = t.stride(0);
    need(t.stride(1) == 1 || K <= 1);
    return {address<const void>(t), rows, K, rows > 1 ? ld : std::max(ld, K)};
}

const at::Tensor& matrix(PyObject* o) {
    const at::Tensor& t = tensor(o);
    need(t.dim() == 2);
    return t;
}
uint8_t* bytes(PyObject* o, int64_t rows, int64_t cols) {  // an output array of codes, scales or words
    const at::Tensor& t = matrix(o);
    need(t.scalar_type() == at::kByte && t.size(0) == rows && t.size(1) == cols && t.is_contiguous());
    return address(t);
}

mx_dtype_t out_type(PyObject* o) {
    if (PyUnicode_CheckExact(o)) {
        if (PyUnicode_CompareWithASCIIString(o, "bf16") == 0) return MX_OUT_BF16;
        need(PyUnicode_CompareWithASCIIString(o, "f32") == 0 || PyUnicode_CompareWithASCIIString(o, "fp32") == 0);
        return MX_OUT_F32;
    }
    const at::ScalarType s = reinterpret_cast<THPDtype*>(o)->scalar_type;
    need(s == at::kFloat || s == at::kBFloat16);
    return s == at::kFloat ? MX_OUT_F32 : MX_OUT_BF16;
}
struct Out {  // an output matrix
    mx_dtype_t type;
    void* data;
    int64_t ld;
};
Out out_matrix(PyObject* type, PyObject* o, int64_t rows, int64_t cols) {
    const mx_dtype_t code = out_type(type);
    const at::Tensor& t = matrix(o);
    need(t.scalar_type() == (code == MX_OUT_F32 ? at::kFloat : at::kBFloat16) && t.size(0) == rows && t.size(1) == cols);
    need(t.stride(1) == 1 || cols <= 1);
    return {code, address<void>(t), rows > 1 ? t.stride(0) : std::max(t.stride(0), cols)};
}

int64_t integer(PyObject* o) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        throw Declined();
    }
    return v;
}
template <int N>
int name_of(PyObject* o, const char* const (&names)[N]) {
    for (int i = 0; i < N; ++i)
        if (PyUnicode_CompareWithASCIIString(o, names[i]) == 0) return i;
    throw Declined();
}
mx_rule_t rule(PyObject* o) {
    static const char* const kNames[] = {"ocp", "floor", "oas"};  // MX_RULE_OCP, MX_RULE_FLOOR, MX_RULE_OAS
    return (mx_rule_t)name_of(o, kNames);
}
mx_elem_t elem(PyObject* o) {
    static const char* const kNames[] = {"e2m1", "e4m3", "e5m2", "e2m3", "e3m2"};
    return (mx_elem_t)name_of(o, kNames);
}
int64_t code_bytes(mx_elem_t e, int64_t K) { return e == MX_ELEM_E2M3 || e == MX_ELEM_E3M2 ? K * 3 / 4 : K; }
bool flag(PyObject* o) { return o == Py_True; }

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Whether the arguments have the types that are served: t = tensor, o = tensor or None, s = text, d = text or torch dtype, i = int,
// b = bool.  Looked at before anything that throws: an exception costs 2 us, a third of the call that the binding's Python code then makes.
bool served(PyObject* const* a, Py_ssize_t n, const char* kinds) {
    for (Py_ssize_t i = 0; i < n; ++i) {
        bool ok = false;
        switch (kinds[i]) {
            case 'o': ok = a[i] == Py_None || THPVariable_CheckExact(a[i]); break;
            case 't': ok = THPVariable_CheckExact(a[i]); break;
            case 's': ok = PyUnicode_CheckExact(a[i]); break;
            case 'd': ok = PyUnicode_CheckExact(a[i]) || THPDtype_Check(a[i]); break;
            case 'i': ok = PyLong_CheckExact(a[i]); break;
            case 'b': ok = PyBool_Check(a[i]); break;
        }
        if (!ok) return false;
    }
    return true;
}

// Runs a call's marshalling; the entry point itself runs without the interpreter's lock, as it did through ctypes.
template <typename F>
PyObject* run(PyObject* const* a, Py_ssize_t n, const char* kinds, F&& marshal) {
    if (n == (Py_ssize_t)strlen(kinds) && served(a, n, kinds) && !at::impl::torch_function_mode_enabled()) {
        try {
            auto call = marshal();
            // (noexcept: an exception out of the C entry point would leave here without the lock)
            const int status = [&]() noexcept {
                int st;
                Py_BEGIN_ALLOW_THREADS
                st = call();
                Py_END_ALLOW_THREADS
                return st;
            }();
            return PyLong_FromLong(status);
        } catch (...) {  // declined, or a tensor that has no address: nothing has been called
        }
    }
    Py_RETURN_NONE;
}

#define MX_CALL(name) PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n)

MX_CALL(quantize) {  // x, rule, codes, scales
    return run(a, n, "tstt", [&] {
        const Rows x = bf16_rows(a[0]);
        const mx_rule_t r = rule(a[1]);
        uint8_t *c = bytes(a[2], x.rows, x.K / 2), *s = bytes(a[3], x.rows, x.K / 32);
        void* st = stream();
        return [=] { return calls.quantize(x.data, x.rows, x.K, x.ld, r, c, s, st); };
    });
}
MX_CALL(quantize_mbs) {  // x, rule, codes, scales, mbs
    return run(a, n, "tsttt", [&] {
        const Rows x = bf16_rows(a[0]);
        const mx_rule_t r = rule(a[1]);
        uint8_t *c = bytes(a[2], x.rows, x.K / 2), *s = bytes(a[3], x.rows, x.K / 32), *m = bytes(a[4], x.rows, (x.K + 127) / 128);
        void* st = stream();
        return [=] { return calls.quantize_mbs(x.data, x.rows, x.K, x.ld, r, c, s, m, st); };
    });
}
MX_CALL(quantize_mbs_pair) {  // x0, x1, rule, codes0, scales0, mbs0, codes1, scales1, mbs1
    return run(a, n, "ttstttttt", [&] {
        const Rows x = bf16_rows(a[0]), y = bf16_rows(a[1]);
        need(x.K == y.K);
        const mx_rule_t r = rule(a[2]);
        uint8_t *c0 = bytes(a[3], x.rows, x.K / 2), *s0 = bytes(a[4], x.rows, x.K / 32), *m0 = bytes(a[5], x.rows, (x.K + 127) / 128);
        uint8_t *c1 = bytes(a[6], y.rows, y.K / 2), *s1 = bytes(a[7], y.rows, y.K / 32), *m1 = bytes(a[8], y.rows, (y.K + 127) / 128);
        void* st = stream();
        return [=] { return calls.quantize_mbs_pair(x.data, x.rows, x.ld, c0, s0, m0, y.data, y.rows, y.ld, c1, s1, m1, x.K, r, st); };
    });
}
MX_CALL(quantize_mbs_dynamic) {  // x, rule, first, count, stride, codes, scales, mbs
    return run(a, n, "tsiiittt", [&] {
        const Rows x = bf16_rows(a[0]);
        const mx_rule_t r = rule(a[1]);
        const int64_t first = integer(a[2]), count = integer(a[3]), stride = integer(a[4]);
        need(first == (int32_t)first && count == (int32_t)count && stride == (int32_t)stride);
        uint8_t *c = bytes(a[5], x.rows, x.K / 2), *s = bytes(a[6], x.rows, x.K / 32), *m = bytes(a[7], x.rows, (x.K + 127) / 128);
        void* st = stream();
        return [=] { return calls.quantize_mbs_dynamic(x.data, x.rows, x.K, x.ld, r, (int32_t)first, (int32_t)count, (int32_t)stride, c, s, m, st); };
    });
}
MX_CALL(quantize_elem) {  // x, elem, rule, use_mbs, codes, scales, mbs (looked at with use_mbs only)
    return run(a, n, "tssbtto", [&] {
        const Rows x = bf16_rows(a[0]);
        const mx_elem_t e = elem(a[1]);
        const mx_rule_t r = rule(a[2]);
        const bool words = flag(a[3]);
        uint8_t *c = bytes(a[4], x.rows, code_bytes(e, x.K)), *s = bytes(a[5], x.rows, x.K / 32), *m = words ? bytes(a[6], x.rows, (x.K + 127) / 128) : nullptr;
        void* st = stream();
        return [=] { return calls.quantize_elem(e, x.data, x.rows, x.K, x.ld, r, words, c, s, m, st); };
    });
}
MX_CALL(dequantize) {  // codes, scales, mbs, type, out
    return run(a, n, "toodt", [&] {
        const at::Tensor& c = matrix(a[0]);
        const int64_t rows = c.size(0), K = c.size(1) * 2;
        const uint8_t *s = optional(a[1]), *m = optional(a[2]), *cp = address(c);
        const Out o = out_matrix(a[3], a[4], rows, K);
        void* st = stream();
        return [=] { return calls.dequantize(cp, s, m, rows, K, o.type, o.data, o.ld, st); };
    });
}

struct Operands {  // MXFP4 operands of a GEMM
    const uint8_t *ac, *as, *am, *bc, *bs, *bm;
    int64_t M, N, K;  // (N: the rows of B)
};
Operands operands(PyObject* ac, PyObject* as, PyObject* am, PyObject* bc, PyObject* bs, PyObject* bm) {
    const at::Tensor &x = matrix(ac), &w = matrix(bc);
    need(x.size(1) == w.size(1));
    return {address(x), optional(as), optional(am), address(w), optional(bs), optional(bm), x.size(0), w.size(0), x.size(1) * 2};
}
MX_CALL(gemm) {  // a_codes, a_scales, b_codes, b_scales, type, out
    return run(a, n, "totodt", [&] {
        const Operands p = operands(a[0], a[1], Py_None, a[2], a[3], Py_None);
        const Out o = out_matrix(a[4], a[5], p.M, p.N);
        void* st = stream();
        return [=] { return calls.gemm(p.ac, p.as, p.bc, p.bs, p.M, p.N, p.K, o.type, o.data, o.ld, st); };
    });
}
MX_CALL(gemm_mbs) {  // a_codes, a_scales, a_mbs, b_codes, b_scales, b_mbs, type, out
    return run(a, n, "tootoodt", [&] {
        const Operands p = operands(a[0], a[1], a[2], a[3], a[4], a[5]);
        const Out o = out_matrix(a[6], a[7], p.M, p.N);
        void* st = stream();
        return [=] { return calls.gemm_mbs(p.ac, p.as, p.am, p.bc, p.bs, p.bm, p.M, p.N, p.K, o.type, o.data, o.ld, st); };
    });
}
struct Groups {
    const int64_t* offsets;
    int32_t count;
};
Groups groups(PyObject* offsets, PyObject* N, int64_t b_rows) {
    const at::Tensor& t = tensor(offsets);
    need(t.scalar_type() == at::kLong && t.is_contiguous());
    const int64_t count = t.numel() - 1;
    int64_t rows;
    need(count == (int32_t)count && !__builtin_mul_overflow(count, integer(N), &rows) && rows == b_rows);
    return {address<const int64_t>(t), (int32_t)count};
}
MX_CALL(gemm_mbs_grouped) {  // a_codes, a_scales, a_mbs, b_codes, b_scales, b_mbs, row_offsets, N, type, out
    return run(a, n, "tootootidt", [&] {
        const Operands p = operands(a[0], a[1], a[2], a[3], a[4], a[5]);
        const Groups g = groups(a[6], a[7], p.N);
        const int64_t N = integer(a[7]);
        const Out o = out_matrix(a[8], a[9], p.M, N);
        void* st = stream();
        return [=] { return calls.gemm_mbs_grouped(p.ac, p.as, p.am, p.bc, p.bs, p.bm, g.count, g.offsets, p.M, N, p.K, o.type, o.data, o.ld, st); };
    });
}
MX_CALL(gemm_mbs_quantize_a) {  // a, rule, a_use_mbs, b_codes, b_scales, b_mbs, type, out
    return run(a, n, "tsbtoodt", [&] {
        const Rows x = bf16_rows(a[0]);
        const mx_rule_t r = rule(a[1]);
        const bool words = flag(a[2]);
        const at::Tensor& w = matrix(a[3]);
        need(w.size(1) * 2 == x.K);
        const uint8_t *bc = address(w), *bs = optional(a[4]), *bm = optional(a[5]);
        const int64_t N = w.size(0);
        const Out o = out_matrix(a[6], a[7], x.rows, N);
        void* st = stream();
        return [=] { return calls.gemm_mbs_quantize_a(x.data, x.ld, r, words, bc, bs, bm, x.rows, N, x.K, o.type, o.data, o.ld, st); };
    });
}
struct ElemOperands {
    mx_elem_t ae, be;
    Operands p;
};
ElemOperands elem_operands(PyObject* const* a) {  // a_elem, a_codes, a_scales, a_mbs, b_elem, b_codes, b_scales, b_mbs
    ElemOperands q;
    q.ae = elem(a[0]);
    q.be = elem(a[4]);
    const at::Tensor &x = matrix(a[1]), &xs = matrix(a[2]), &w = matrix(a[5]), &ws = matrix(a[6]);
    const int64_t K = xs.size(1) * 32;
    need(ws.size(1) * 32 == K && x.size(1) == code_bytes(q.ae, K) && w.size(1) == code_bytes(q.be, K));
    q.p = {address(x), address(xs), optional(a[3]), address(w), address(ws), optional(a[7]), x.size(0), w.size(0), K};
    return q;
}
MX_CALL(gemm_mbs_elem) {  // a_elem .. b_mbs, type, out
    return run(a, n, "sttosttodt", [&] {
        const ElemOperands q = elem_operands(a);
        const Out o = out_matrix(a[8], a[9], q.p.M, q.p.N);
        void* st = stream();
        return [=] {
            const Operands& p = q.p;
            return calls.gemm_mbs_elem(q.ae, p.ac, p.as, p.am, q.be, p.bc, p.bs, p.bm, p.M, p.N, p.K, o.type, o.data, o.ld, st);
        };
    });
}
MX_CALL(gemm_mbs_elem_grouped) {  // a_elem .. b_mbs, row_offsets, N, type, out
    return run(a, n, "sttosttotidt", [&] {
        const ElemOperands q = elem_operands(a);
        const Groups g = groups(a[8], a[9], q.p.N);
        const int64_t N = integer(a[9]);
        const Out o = out_matrix(a[10], a[11], q.p.M, N);
        void* st = stream();
        return [=] {
            const Operands& p = q.p;
            return calls.gemm_mbs_elem_grouped(q.ae, p.ac, p.as, p.am, q.be, p.bc, p.bs, p.bm, g.count, g.offsets, p.M, N, p.K, o.type, o.data, o.ld, st);
        };
    });
}

// entry points' addresses, in the order of `Calls`
PyObject* use(PyObject*, PyObject* const* a, Py_ssize_t n) {
    constexpr Py_ssize_t kCount = sizeof(Calls) / sizeof(void*);
    if (n != kCount) {
        PyErr_SetString(PyExc_TypeError, "the address of every entry point is wanted");
        return nullptr;
    }
    void* found[kCount];
    for (Py_ssize_t i = 0; i < kCount; ++i) {
        found[i] = PyLong_AsVoidPtr(a[i]);
        if (!found[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
            return nullptr;
        }
    }
    memcpy(&calls, found, sizeof calls);
    Py_RETURN_NONE;
}

// what this module was compiled against: the binding compares it before any other call (torch's objects are read through inline
// headers, at the offsets of that torch)
PyObject* built_for(PyObject*, PyObject* const*, Py_ssize_t) { return PyUnicode_FromString(MX_BUILT_FOR); }

#define MX_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MX_METHOD(built_for), MX_METHOD(use), MX_METHOD(quantize), MX_METHOD(quantize_mbs), MX_METHOD(quantize_mbs_pair), MX_METHOD(quantize_mbs_dynamic),
                         MX_METHOD(quantize_elem), MX_METHOD(dequantize), MX_METHOD(gemm), MX_METHOD(gemm_mbs), MX_METHOD(gemm_mbs_grouped),
                         MX_METHOD(gemm_mbs_quantize_a), MX_METHOD(gemm_mbs_elem), MX_METHOD(gemm_mbs_elem_grouped), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
