// The calls of api.py that a serving loop makes, from tensors to the C ABI in one step.
//
// At decode a kernel runs for five to ten microseconds, and marshalling its arguments in Python (attribute
// checks, a ctypes object per argument, the current stream, the workspace query) took as long again: a
// 1024 x 1024 linear at 16 rows cost 10.7 us of host time per call for 5.5 us of GPU time.  Each function
// here checks its tensors, asks the allocator for an output if none was given, takes PyTorch's current
// stream and calls the entry point, whose address comes from the library the caller loaded (so that a
// second build of the library can be called through the same code).
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/milo.h"

namespace {

// The entry points of one loaded library.
struct Entries {
    decltype(&milo_w3_packed_bytes) packed_bytes;
    decltype(&milo_pack_w3) pack;
    decltype(&milo_pack_w3_sym) pack_sym;
    decltype(&milo_w3lr_gemm_workspace) gemm_workspace;
    decltype(&milo_w3lr_gemm_flags) gemm;
    decltype(&milo_workspace_init) workspace_init;
    decltype(&milo_moe_w3lr_workspace) moe_workspace;
    decltype(&milo_moe_w3lr_forward_flags) moe;
};
constexpr const char* kEntryNames[] = {"milo_w3_packed_bytes", "milo_pack_w3", "milo_pack_w3_sym",
                                       "milo_w3lr_gemm_workspace", "milo_w3lr_gemm_flags", "milo_workspace_init",
                                       "milo_moe_w3lr_workspace", "milo_moe_w3lr_forward_flags"};
constexpr size_t kEntries = sizeof(kEntryNames) / sizeof(kEntryNames[0]);
static_assert(sizeof(Entries) == kEntries * sizeof(void*), "one address per entry point");

void* current_stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

// A contiguous GPU tensor of type `dt`, or nullptr with a TypeError set.
const at::Tensor* device_tensor(PyObject* o, at::ScalarType dt, const char* name) {
    if (THPVariable_Check(o)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (t.is_cuda() && t.scalar_type() == dt && t.is_contiguous()) return &t;
    }
    PyErr_Format(PyExc_TypeError, "%s must be a contiguous CUDA tensor of torch.%s", name,
                 dt == at::kHalf ? "float16" : dt == at::kBFloat16 ? "bfloat16" : dt == at::kInt ? "int32" : "float32");
    return nullptr;
}
// Any tensor's address (nullptr for None), as api.py's pointers.
bool address(PyObject* o, const char* name, void** p) {
    *p = nullptr;
    if (o == Py_None) return true;
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
        return false;
    }
    *p = THPVariable_Unpack(o).data_ptr();
    return true;
}
bool whole(PyObject* o, int64_t* v) {
    *v = PyLong_AsLongLong(o);
    return !(*v == -1 && PyErr_Occurred());
}

// at::Tensor calls throw C++ exceptions; they become the Python exceptions that PyTorch's own calls raise
// (torch.OutOfMemoryError from an allocation, for one).
template <typename F>
PyObject* guarded(F&& f) {
    HANDLE_TH_ERRORS
    return f();
    END_HANDLE_TH_ERRORS
}
PyObject* status_object(int st) { return PyLong_FromLong(st); }

// entries(dict name -> address) -> capsule for the functions below
void free_entries(PyObject* c) { delete static_cast<Entries*>(PyCapsule_GetPointer(c, "milo.entries")); }
PyObject* py_entries(PyObject*, PyObject* dict) {
    void* addr[kEntries];
    for (size_t i = 0; i < kEntries; ++i) {
        PyObject* v = PyDict_Check(dict) ? PyDict_GetItemString(dict, kEntryNames[i]) : nullptr;
        addr[i] = v ? PyLong_AsVoidPtr(v) : nullptr;
        if (!addr[i]) {
            if (!PyErr_Occurred()) PyErr_Format(PyExc_ValueError, "no address of %s", kEntryNames[i]);
            return nullptr;
        }
    }
    Entries* e = new Entries;
    memcpy(static_cast<void*>(e), addr, sizeof(Entries));
    return PyCapsule_New(e, "milo.entries", free_entries);
}
const Entries* entries_of(PyObject* c) { return static_cast<const Entries*>(PyCapsule_GetPointer(c, "milo.entries")); }

// gemm(entries, X, q3, U, V, N, K, r, flags, out, workspace): the output tensor, or a non-zero status.  U None
// means rank 0, r None the number of U's columns.
PyObject* py_gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 11) return PyErr_Format(PyExc_TypeError, "gemm takes 11 arguments");
    return guarded([&]() -> PyObject* {
        const Entries* e = entries_of(a[0]);
        if (!e) return nullptr;
        const bool bf = THPVariable_Check(a[1]) && THPVariable_Unpack(a[1]).scalar_type() == at::kBFloat16;
        const at::Tensor* X = device_tensor(a[1], bf ? at::kBFloat16 : at::kHalf, "X");
        if (!X) return nullptr;
        if (X->dim() != 2) return PyErr_Format(PyExc_ValueError, "X must have two dimensions");
        int64_t N, K, r, flags;
        if (!whole(a[5], &N) || !whole(a[6], &K) || !whole(a[8], &flags)) return nullptr;
        if (a[3] == Py_None) r = 0;
        else if (a[7] != Py_None) { if (!whole(a[7], &r)) return nullptr; }
        else if (THPVariable_Check(a[3]) && THPVariable_Unpack(a[3]).dim() == 2) r = THPVariable_Unpack(a[3]).size(1);
        else return PyErr_Format(PyExc_TypeError, "U must be a matrix");
        const int64_t M = X->size(0);
        if (X->size(1) != K) return PyErr_Format(PyExc_ValueError, "X and weight disagree on K");
        if (a[3] != Py_None && !(flags & MILO_LR_INT3) && THPVariable_Check(a[3]) &&
            THPVariable_Unpack(a[3]).scalar_type() != X->scalar_type())
            return PyErr_Format(PyExc_TypeError, "the compensator and the activations must have the same 16-bit type");
        void *q3, *U, *V, *Y, *ws;
        if (!address(a[2], "q3", &q3) || !address(a[3], "U", &U) || !address(a[4], "V", &V) || !address(a[9], "out", &Y) ||
            !address(a[10], "workspace", &ws))
            return nullptr;
        void* const stream = current_stream();
        at::Tensor out, own;
        if (a[9] == Py_None) {
            out = at::empty({M, N}, X->options());
            Y = out.data_ptr();
        }
        size_t ws_bytes;
        if (a[10] == Py_None) {
            const size_t need = e->gemm_workspace(M, N, K, (int)r);
            own = at::empty({(int64_t)(need > 256 ? need : 256)}, X->options().dtype(at::kByte));
            ws = own.data_ptr();
            ws_bytes = (size_t)own.numel();
            // Only the state has to start at zero; what lies behind may hold anything.
            const int st = e->workspace_init(ws, ws_bytes < MILO_WORKSPACE_STATE_BYTES ? ws_bytes : MILO_WORKSPACE_STATE_BYTES, stream);
            if (st != MILO_OK) return status_object(st);
        } else {
            ws_bytes = (size_t)THPVariable_Unpack(a[10]).numel();
        }
        const unsigned f = (unsigned)flags | (bf ? MILO_ACT_BF16 : 0u);
        const milo_half* x = static_cast<const milo_half*>(X->data_ptr());
        int st;
        Py_BEGIN_ALLOW_THREADS
        st = e->gemm(x, M, N, K, q3, U, V, (int)r, f, static_cast<milo_half*>(Y), ws, ws_bytes, stream);
        Py_END_ALLOW_THREADS
        if (st != MILO_OK) return status_object(st);
        if (a[9] == Py_None) return THPVariable_Wrap(std::move(out));
        Py_INCREF(a[9]);
        return a[9];
    });
}

// moe(entries, X, ids, gates, table, H, F, E, r_max, flags, out, workspace, own): the output tensor, a
// non-zero status, or, where `own` is true and the workspace is missing or too small for this call, minus
// the bytes it needs.
PyObject* py_moe(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 13) return PyErr_Format(PyExc_TypeError, "moe takes 13 arguments");
    return guarded([&]() -> PyObject* {
        const Entries* e = entries_of(a[0]);
        if (!e) return nullptr;
        int64_t H, F, E, r_max, flags;
        if (!whole(a[5], &H) || !whole(a[6], &F) || !whole(a[7], &E) || !whole(a[8], &r_max) || !whole(a[9], &flags))
            return nullptr;
        const at::Tensor* X = device_tensor(a[1], (flags & MILO_ACT_BF16) ? at::kBFloat16 : at::kHalf, "X");
        const at::Tensor* ids = X ? device_tensor(a[2], at::kInt, "ids") : nullptr;
        const at::Tensor* gates = ids ? device_tensor(a[3], at::kFloat, "gates") : nullptr;
        if (!gates) return nullptr;
        if (X->dim() != 2 || ids->dim() != 2) return PyErr_Format(PyExc_ValueError, "X and ids must have two dimensions");
        const int64_t T = X->size(0), topk = ids->size(1);
        // The kernels go by H and T alone: rows of another width would be multiplied with the experts' [F x H] weights at the
        // wrong stride, wider ones past the weights' end, and missing ids or gates would be read past the end of theirs.
        if (X->size(1) != H) return status_object(X->size(1) > H ? MILO_ERR_WORKSPACE : MILO_ERR_SHAPE);
        if (ids->size(0) < T || gates->numel() < T * topk)
            return PyErr_Format(PyExc_ValueError, "ids and gates must have a row for every row of X");
        void *table, *Y, *ws;
        if (!address(a[4], "table", &table) || !address(a[10], "out", &Y) || !address(a[11], "workspace", &ws)) return nullptr;
        const size_t have = a[11] == Py_None ? 0 : (size_t)THPVariable_Unpack(a[11]).numel();
        if (a[12] == Py_True) {
            const size_t need = e->moe_workspace(T, H, F, (int)E, (int)topk, (int)r_max);
            if (!ws || have < need) return PyLong_FromLongLong(-(long long)(need > 256 ? need : 256));
        }
        at::Tensor out;
        if (a[10] == Py_None) {
            out = at::empty({T, H}, X->options());
            Y = out.data_ptr();
        }
        void* const stream = current_stream();
        const milo_half* x = static_cast<const milo_half*>(X->data_ptr());
        const int32_t* id = static_cast<const int32_t*>(ids->data_ptr());
        const float* gate = static_cast<const float*>(gates->data_ptr());
        int st;
        Py_BEGIN_ALLOW_THREADS
        st = e->moe(x, T, H, F, static_cast<const milo_w3lr_expert*>(table), (int)E, (int)r_max, id, gate, (int)topk,
                    (unsigned)flags, static_cast<milo_half*>(Y), ws, have, stream);
        Py_END_ALLOW_THREADS
        if (st != MILO_OK) return status_object(st);
        if (a[10] == Py_None) return THPVariable_Wrap(std::move(out));
        Py_INCREF(a[10]);
        return a[10];
    });
}

// pack(entries, W, group_size, symmetric): the blob of W, or a non-zero status.
PyObject* py_pack(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 4) return PyErr_Format(PyExc_TypeError, "pack takes 4 arguments");
    return guarded([&]() -> PyObject* {
        const Entries* e = entries_of(a[0]);
        if (!e) return nullptr;
        const at::Tensor* W = device_tensor(a[1], at::kFloat, "W");
        int64_t group;
        if (!W || !whole(a[2], &group)) return nullptr;
        if (W->dim() != 2) return PyErr_Format(PyExc_ValueError, "W must have two dimensions");
        const int symmetric = PyObject_IsTrue(a[3]);
        if (symmetric < 0) return nullptr;
        const int64_t N = W->size(0), K = W->size(1);
        const size_t bytes = e->packed_bytes(N, K);             // (0 for a shape the call below refuses)
        at::Tensor q3 = at::empty({(int64_t)(bytes > 16 ? bytes : 16)}, W->options().dtype(at::kByte));
        void* const stream = current_stream();
        const float* w = static_cast<const float*>(W->data_ptr());
        void* const q = q3.data_ptr();
        int st;
        Py_BEGIN_ALLOW_THREADS
        st = (symmetric ? e->pack_sym : e->pack)(w, N, K, (int)group, q, stream);
        Py_END_ALLOW_THREADS
        if (st != MILO_OK) return status_object(st);
        return THPVariable_Wrap(std::move(q3));
    });
}

PyMethodDef kMethods[] = {
    {"entries", py_entries, METH_O, "addresses of a loaded library's entry points"},
    {"gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(py_gemm)), METH_FASTCALL, "milo_w3lr_gemm_flags on tensors"},
    {"moe", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(py_moe)), METH_FASTCALL, "milo_moe_w3lr_forward_flags on tensors"},
    {"pack", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(py_pack)), METH_FASTCALL, "milo_pack_w3(_sym) on tensors"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_milo_torch", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__milo_torch(void) { return PyModule_Create(&kModule); }
