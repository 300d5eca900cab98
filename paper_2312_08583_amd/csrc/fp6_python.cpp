// Marshalling of the hot-path calls for Python: the same checks as binding.py makes, on the tensors themselves.
//
// A call from Python took 10 us, of which the kernel of a small layer is 3: some thirty attribute reads and checks, a ctypes call with
// eleven conversions and the look-up of the current stream.  With them here it takes 3.3 to 4.4, most of it the launch (1 x 1024 x 1024,
// calls back to back 10.3 -> 4.7 us; the four calls of a 7B-shaped block at four rows 50 -> 39).  Whatever is not a plain call - a
// missing workspace, a tensor subclass, an active function or dispatch mode (torch.set_default_device installs one for good), a wrapped
// tensor, an argument that does not fit - gets None, and binding.py takes the call from there: it allocates, and it words the errors.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/fp6_linear.h"

namespace {

// the entry points of the loaded library, as binding.py found them
decltype(&fp6_linear) call_linear;
decltype(&fp6_linear_variant) call_variant;
decltype(&fp6_linear_fgq) call_fgq;
decltype(&fp5_linear) call_fp5;
decltype(&fp6_linear_v2) call_v2;
decltype(&fp6_linear_v2_bf16) call_v2_bf16;
decltype(&fp6_linear_group) call_group;
decltype(&fp6_linear_workspace_bytes) need_linear;
decltype(&fp6_linear_variant_workspace_bytes) need_variant;
decltype(&fp6_linear_fgq_workspace_bytes) need_fgq;
decltype(&fp5_linear_workspace_bytes) need_fp5;
decltype(&fp6_linear_v2_workspace_bytes) need_v2;          // of both plane-layout-2 calls
decltype(&fp6_linear_group_workspace_bytes) need_group;
PyObject* fail = nullptr;          // fail(status, name) raises

enum Kind { kLinear, kVariant, kFgq, kFp5, kV2, kV2Bf16, kKinds };
constexpr const char* kNames[kKinds] = {"fp6_linear", "fp6_linear_variant", "fp6_linear_fgq", "fp5_linear", "fp6_linear_v2",
                                        "fp6_linear_v2_bf16"};

bool modes_active()
{
    return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set();
}

// A plain contiguous device tensor of this type, or nullptr.
const at::Tensor* plain(PyObject* o, c10::ScalarType type)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || t.layout() != c10::kStrided || !t.is_contiguous()) return nullptr;
    const c10::DispatchKeySet keys = t.key_set();
    if (keys.has(c10::DispatchKey::Python) || keys.has(c10::DispatchKey::FuncTorchBatched) ||
        keys.has(c10::DispatchKey::FuncTorchGradWrapper) || keys.has(c10::DispatchKey::Functionalize))
        return nullptr;
    return &t;
}

bool whole(PyObject* o, int64_t* v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return !overflow;
}

struct Layer {
    const void *x, *hi, *lo, *scales;
    void* y;
    int64_t M, N, K;
    const at::Tensor* X;
};

// X, planes, scales, N and K, each checked against the sizes that the others imply.
bool read_layer(PyObject* X, PyObject* hi, PyObject* lo, PyObject* scales, PyObject* n, PyObject* k, int64_t block, int64_t lo_div,
                c10::ScalarType type, Layer* l)
{
    if (!whole(n, &l->N) || !whole(k, &l->K)) return false;
    const int64_t N = l->N, K = l->K;
    if (N <= 0 || K <= 0 || N % FP6_TILE || K % FP6_TILE || N > (int64_t)1 << 30 || K > (int64_t)1 << 30) return false;
    if (block && (block < 0 || K % block)) return false;
    const at::Tensor *x = plain(X, type), *h = plain(hi, c10::kByte), *o = plain(lo, c10::kByte), *s = plain(scales, c10::kHalf);
    if (!x || !h || !o || !s || x->dim() != 2 || x->size(1) != K || x->size(0) < 1) return false;
    if (h->numel() != N * K / 2 || o->numel() != N * K / lo_div || s->numel() != N * (block ? K / block : 1)) return false;
    l->M = x->size(0);
    l->x = x->data_ptr();
    l->hi = h->data_ptr();
    l->lo = o->data_ptr();
    l->scales = s->data_ptr();
    l->X = x;
    return true;
}

bool read_out(PyObject* out, c10::ScalarType type, Layer* l)
{
    const at::Tensor* y = plain(out, type);
    if (!y || y->dim() != 2 || y->size(0) != l->M || y->size(1) != l->N) return false;
    l->y = y->data_ptr();
    return true;
}

// linear(kind, X, hi, lo, scales, N, K, block, out, workspace, variant, split_k) -> Y, or None
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t count)
{
    int64_t kind, block, variant, split_k;
    if (count != 12 || !fail || !whole(a[0], &kind) || kind < 0 || kind >= kKinds || !whole(a[7], &block) || !whole(a[10], &variant) ||
        !whole(a[11], &split_k) || variant != (int)variant || split_k != (int)split_k || modes_active())
        Py_RETURN_NONE;
    PyObject* result = nullptr;
    int status = FP6_OK;
    try {
        const c10::ScalarType type = kind == kV2Bf16 ? c10::kBFloat16 : c10::kHalf;
        Layer l;
        if (!read_layer(a[1], a[2], a[3], a[4], a[5], a[6], block, kind == kFp5 ? 8 : 4, type, &l)) Py_RETURN_NONE;
        if (kind == kFgq && block <= 0) Py_RETURN_NONE;
        const at::Tensor* ws = nullptr;
        if (a[9] == Py_None) {
            // a call that needs no workspace; one that does has it allocated by binding.py
            const int v = (int)variant, d = (int)split_k;
            const size_t need = kind == kLinear    ? need_linear(l.M, l.N, l.K)
                                : kind == kVariant ? need_variant(l.M, l.N, l.K, v, d)
                                : kind == kFgq     ? need_fgq(l.M, l.N, l.K, block, v, d)
                                : kind == kFp5     ? need_fp5(l.M, l.N, l.K, v, d)
                                                   : need_v2(l.M, l.N, l.K, v, d);
            if (need) Py_RETURN_NONE;
        } else {
            ws = plain(a[9], c10::kByte);
            if (!ws) Py_RETURN_NONE;
        }
        if (a[8] == Py_None) {
            const at::Tensor y = at::empty({l.M, l.N}, l.X->options());
            l.y = y.data_ptr();
            result = THPVariable_Wrap(y);
            if (!result) return nullptr;
        } else {
            if (!read_out(a[8], type, &l)) Py_RETURN_NONE;
            result = a[8];
            Py_INCREF(result);
        }
        void* w = ws ? ws->data_ptr() : nullptr;
        const size_t bytes = ws ? (size_t)ws->numel() : 0;
        void* stream = c10::hip::getCurrentHIPStream().stream();
        const uint16_t *x = (const uint16_t*)l.x, *s = (const uint16_t*)l.scales;
        uint16_t* y = (uint16_t*)l.y;
        Py_BEGIN_ALLOW_THREADS
        switch (kind) {
            case kLinear: status = call_linear(x, l.M, l.hi, l.lo, s, l.N, l.K, y, w, bytes, stream); break;
            case kVariant: status = call_variant(x, l.M, l.hi, l.lo, s, l.N, l.K, y, w, bytes, stream, (int)variant, (int)split_k); break;
            case kFgq: status = call_fgq(x, l.M, l.hi, l.lo, s, l.N, l.K, block, y, w, bytes, stream, (int)variant, (int)split_k); break;
            case kFp5: status = call_fp5(x, l.M, l.hi, l.lo, s, l.N, l.K, y, w, bytes, stream, (int)variant, (int)split_k); break;
            case kV2: status = call_v2(x, l.M, l.hi, l.lo, s, l.N, l.K, y, w, bytes, stream, (int)variant, (int)split_k); break;
            default: status = call_v2_bf16(x, l.M, l.hi, l.lo, s, l.N, l.K, y, w, bytes, stream, (int)variant, (int)split_k);
        }
        Py_END_ALLOW_THREADS
    } catch (...) {
        Py_XDECREF(result);          // (the allocation of Y threw, or the look-up of the stream behind it)
        Py_RETURN_NONE;
    }
    if (status == FP6_OK) return result;
    Py_DECREF(result);
    return PyObject_CallFunction(fail, "is", status, kNames[kind]);
}

// group(layers, outs, workspace) -> list of Y, or None
PyObject* group(PyObject*, PyObject* const* a, Py_ssize_t count)
{
    if (count != 3 || !fail || modes_active()) Py_RETURN_NONE;
    auto sequence = [](PyObject* o) { return PyList_CheckExact(o) || PyTuple_CheckExact(o); };
    if (!sequence(a[0]) || !sequence(a[1])) Py_RETURN_NONE;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(a[0]);
    if (n < 1 || n > FP6_GROUP_MAX || PySequence_Fast_GET_SIZE(a[1]) < n) Py_RETURN_NONE;
    fp6_linear_problem problems[FP6_GROUP_MAX];
    PyObject* ys[FP6_GROUP_MAX];
    int status = FP6_OK;
    try {
        int64_t M = 0;
        for (Py_ssize_t i = 0; i < n; i++) {
            PyObject* p = PySequence_Fast_GET_ITEM(a[0], i);
            ys[i] = PySequence_Fast_GET_ITEM(a[1], i);
            Layer l;
            if (!sequence(p) || PySequence_Fast_GET_SIZE(p) != 6) Py_RETURN_NONE;
            PyObject** f = PySequence_Fast_ITEMS(p);
            if (!read_layer(f[0], f[1], f[2], f[3], f[4], f[5], 0, 4, c10::kHalf, &l) || (i && l.M != M) || !read_out(ys[i], c10::kHalf, &l))
                Py_RETURN_NONE;
            M = l.M;
            problems[i] = fp6_linear_problem{(const uint16_t*)l.x, l.hi, l.lo, (const uint16_t*)l.scales, l.N, l.K, (uint16_t*)l.y};
        }
        const at::Tensor* ws = nullptr;
        if (a[2] == Py_None) {
            if (need_group(M, problems, (int)n)) Py_RETURN_NONE;
        } else {
            ws = plain(a[2], c10::kByte);
            if (!ws) Py_RETURN_NONE;
        }
        void* w = ws ? ws->data_ptr() : nullptr;
        const size_t bytes = ws ? (size_t)ws->numel() : 0;
        void* stream = c10::hip::getCurrentHIPStream().stream();
        for (Py_ssize_t i = 0; i < n; i++) Py_INCREF(ys[i]);          // (the lists may change while other threads run)
        Py_BEGIN_ALLOW_THREADS
        status = call_group(M, problems, (int)n, w, bytes, stream);
        Py_END_ALLOW_THREADS
    } catch (...) {
        Py_RETURN_NONE;
    }
    PyObject* list = status == FP6_OK ? PyList_New(n) : nullptr;
    for (Py_ssize_t i = 0; i < n; i++) {
        if (list) PyList_SET_ITEM(list, i, ys[i]);
        else Py_DECREF(ys[i]);
    }
    if (status != FP6_OK) return PyObject_CallFunction(fail, "is", status, "fp6_linear_group");
    return list;
}

// bind(address of each entry point in the order of the declarations above, fail)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t count)
{
    if (count != 14) return PyErr_Format(PyExc_TypeError, "bind takes thirteen addresses and a function");
    void* p[13];
    for (int i = 0; i < 13; i++) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    call_linear = (decltype(call_linear))p[0];
    call_variant = (decltype(call_variant))p[1];
    call_fgq = (decltype(call_fgq))p[2];
    call_fp5 = (decltype(call_fp5))p[3];
    call_v2 = (decltype(call_v2))p[4];
    call_v2_bf16 = (decltype(call_v2_bf16))p[5];
    call_group = (decltype(call_group))p[6];
    need_linear = (decltype(need_linear))p[7];
    need_variant = (decltype(need_variant))p[8];
    need_fgq = (decltype(need_fgq))p[9];
    need_fp5 = (decltype(need_fp5))p[10];
    need_v2 = (decltype(need_v2))p[11];
    need_group = (decltype(need_group))p[12];
    Py_INCREF(a[13]);
    PyObject* old = fail;
    fail = a[13];
    Py_XDECREF(old);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"linear", (PyCFunction)(void (*)())linear, METH_FASTCALL, nullptr},
                         {"group", (PyCFunction)(void (*)())group, METH_FASTCALL, nullptr},
                         {"bind", (PyCFunction)(void (*)())bind, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
