// The ordinary calls of binding.py without its Python and ctypes steps: new outputs from torch's allocator, the current stream,
// the cached workspace.  attn() and rmsnorm() do what attn_jvp_fwd_ex and attn_jvp_rmsnorm_fwd of binding.py do for plain
// contiguous GPU tensors that fit together; for anything else (other tensor types, named dimensions, modes that watch torch's calls, functorch's
// wrapped tensors, another current device, calls recorded into a graph, arguments that do not fit) they return None, and binding.py does the whole call,
// errors included.  A call's host time is what bounds small shapes: 13.1 -> 7.1 us a call back to back (8 heads, 300 queries,
// 77 keys, d = 64, whose kernel takes 4.5), 8.5 -> 5.4 for the normalisation; outputs without torch's dispatcher another 0.8 of the former.
#include <Python.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPGraphsC10Utils.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include "../../include/attn_jvp.h"

namespace {

// what binding.py hands over at its first call: entry points of the library it has loaded, its workspace cache, the locks of its entries,
// and the functions that fill both
decltype(&attn_jvp_fwd_ex) fwd_ex;
decltype(&attn_jvp_rmsnorm_fwd) rmsnorm_fwd;
decltype(&attn_jvp_workspace_bytes) bytes_bf16, bytes_fp32;
PyObject *workspaces, *new_workspace, *locks, *new_lock, *name_acquire, *name_release;

PyObject* init(PyObject*, PyObject* args) {
    unsigned long long at[4];
    PyObject *cache, *fill, *cache_locks, *fill_lock;
    if (!PyArg_ParseTuple(args, "KKKKOOOO", &at[0], &at[1], &at[2], &at[3], &cache, &fill, &cache_locks, &fill_lock)) return nullptr;
    if (!name_acquire && !(name_acquire = PyUnicode_InternFromString("acquire"))) return nullptr;
    if (!name_release && !(name_release = PyUnicode_InternFromString("release"))) return nullptr;
    fwd_ex = reinterpret_cast<decltype(fwd_ex)>(at[0]);
    rmsnorm_fwd = reinterpret_cast<decltype(rmsnorm_fwd)>(at[1]);
    bytes_bf16 = reinterpret_cast<decltype(bytes_bf16)>(at[2]);
    bytes_fp32 = reinterpret_cast<decltype(bytes_fp32)>(at[3]);
    const auto keep = [](PyObject*& slot, PyObject* o) {
        Py_INCREF(o);
        Py_XSETREF(slot, o);
    };
    keep(workspaces, cache);
    keep(new_workspace, fill);
    keep(locks, cache_locks);
    keep(new_lock, fill_lock);
    Py_RETURN_NONE;
}

// Nothing is to see or change torch's calls but torch itself.
bool plain_mode() {
    return !at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set() &&
           !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
}
// A torch.Tensor or Parameter that is a plain contiguous array in GPU memory (no subclass, no wrapper, no names for outputs to take over).
const at::Tensor* plain_tensor(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() &&
           !t.key_set().has(c10::DispatchKey::Python) && !t.has_names() && t.is_contiguous() ? &t : nullptr;
}
// at::empty without its way through the dispatcher, 0.3 us each, by torch's internal interface.  What would have a say there has been
// looked for (plain_mode(), plain_tensor()), but for torch.utils.deterministic.fill_uninitialized_memory, whose fill is left out: the
// kernels write every element.
at::Tensor fresh(at::IntArrayRef sizes, at::ScalarType dtype, c10::Device device) {
    return at::Tensor(at::detail::empty_cuda(sizes, dtype, device, std::nullopt));
}
bool fits_int(int64_t n) { return n >= 0 && n <= INT_MAX; }

// Scratch that a shape can use: pure arithmetic on the six numbers, kept for the shapes last seen (under the GIL).
size_t scratch_bytes(int B, int H, int Lq, int Lkv, int d, bool f32) {
    struct Entry { int key[6]; size_t bytes; };
    static Entry seen[64] = {};      // (zeros match no shape: B > 0)
    const int key[6] = {B, H, Lq, Lkv, d, f32};
    unsigned h = 0;
    for (int k : key) h = (h ^ (unsigned)k) * 2654435761u;
    Entry& e = seen[h >> 26];
    for (int i = 0; i < 6; ++i)
        if (e.key[i] != key[i]) {
            e.bytes = (f32 ? bytes_fp32 : bytes_bf16)(B, H, Lq, Lkv, d);
            for (int j = 0; j < 6; ++j) e.key[j] = key[j];
            break;
        }
    return e.bytes;
}

// binding.py's workspace of a device and stream, with its lock held until the object goes: the launches of a call hand the
// workspace on to one another, and another thread's on the same stream must not come between them (the GIL is released
// meanwhile).
class Workspace {
    PyObject *lock = nullptr, *tensor = nullptr;

public:
    // At least `need` bytes; false with a Python error.
    bool take(PyObject* q, hipStream_t stream, size_t need) {
        PyObject* device = PyObject_GetAttrString(q, "device");
        PyObject* raw = device ? PyLong_FromVoidPtr(stream) : nullptr;
        PyObject* key = raw ? PyTuple_Pack(2, device, raw) : nullptr;
        if (key) {
            PyObject* l = PyDict_GetItemWithError(locks, key);      // (borrowed)
            if (l) Py_INCREF(l);
            else if (!PyErr_Occurred()) l = PyObject_CallOneArg(new_lock, key);
            PyObject* got = l ? PyObject_CallMethodNoArgs(l, name_acquire) : nullptr;
            if (got) lock = l;
            else Py_XDECREF(l);
            Py_XDECREF(got);
        }
        if (lock) {
            tensor = PyDict_GetItemWithError(workspaces, key);
            Py_XINCREF(tensor);
            if (!PyErr_Occurred() && (!tensor || (size_t)THPVariable_Unpack(tensor).numel() < need)) {
                Py_CLEAR(tensor);
                PyObject* n = PyLong_FromSize_t(need);
                if (n) tensor = PyObject_CallFunctionObjArgs(new_workspace, device, Py_None, raw, n, nullptr);
                Py_XDECREF(n);
            }
        }
        Py_XDECREF(key);
        Py_XDECREF(raw);
        Py_XDECREF(device);
        return tensor != nullptr;
    }
    const at::Tensor& get() const { return THPVariable_Unpack(tensor); }
    Workspace() = default;
    Workspace(const Workspace&) = delete;
    ~Workspace() {
        if (!lock && !tensor) return;
        PyObject *type, *value, *trace;      // (an error on its way stays)
        PyErr_Fetch(&type, &value, &trace);
        Py_XDECREF(tensor);
        if (lock) {
            PyObject* r = PyObject_CallMethodNoArgs(lock, name_release);
            if (!r) PyErr_WriteUnraisable(lock);
            Py_XDECREF(r);
            Py_DECREF(lock);
        }
        PyErr_Restore(type, value, trace);
    }
};

// attn(q, k, v, tq, tk, tv, scale, out_dtype, kernel, flags, layout, with_workspace) -> (o, to, lse), an error code, or None
PyObject* attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 12 || !fwd_ex || !plain_mode() || !PyFloat_CheckExact(a[6]) || !THPDtype_Check(a[7])) Py_RETURN_NONE;
    const at::Tensor* t[6];
    for (int i = 0; i < 6; ++i) {
        t[i] = i > 2 && a[i] == Py_None ? nullptr : plain_tensor(a[i]);
        if (!t[i] && !(i > 2 && a[i] == Py_None)) Py_RETURN_NONE;
    }
    if ((t[4] == nullptr) != (t[5] == nullptr) || (!t[3] && t[4])) Py_RETURN_NONE;
    const at::Tensor &q = *t[0], &k = *t[1];
    const long kernel = PyLong_AsLong(a[8]), flags = PyLong_AsLong(a[9]), layout = PyLong_AsLong(a[10]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const auto dtype = q.scalar_type();
    const bool f32 = dtype == at::kFloat;
    const auto out_dtype = reinterpret_cast<THPDtype*>(a[7])->scalar_type;
    if ((!f32 && dtype != at::kBFloat16) || (out_dtype != at::kFloat && out_dtype != dtype)) Py_RETURN_NONE;
    if (q.dim() != 4 || k.dim() != 4 || (layout != ATTN_JVP_LAYOUT_BHLD && layout != ATTN_JVP_LAYOUT_BLHD) || !fits_int(kernel) || !fits_int(flags)) Py_RETURN_NONE;
    const int l = layout == ATTN_JVP_LAYOUT_BLHD ? 1 : 2;      // dimension of the rows
    const int64_t B = q.size(0), H = q.size(3 - l), Lq = q.size(l), Lkv = k.size(l), d = q.size(3);
    if (!fits_int(B) || !fits_int(H) || !fits_int(Lq) || !fits_int(Lkv) || !fits_int(d)) Py_RETURN_NONE;
    if (k.size(0) != B || k.size(3 - l) != H || k.size(3) != d) Py_RETURN_NONE;
    for (int i = 1; i < 6; ++i)
        if (t[i] && (t[i]->scalar_type() != dtype || t[i]->device() != q.device() || t[i]->sizes() != (i == 3 ? q : k).sizes())) Py_RETURN_NONE;
    const auto index = q.device().index();
    if (c10::hip::current_device() != index) Py_RETURN_NONE;
    const hipStream_t stream = c10::hip::getCurrentHIPStream(index).stream();
    const size_t need = a[11] == Py_True ? scratch_bytes((int)B, (int)H, (int)Lq, (int)Lkv, (int)d, f32) : 0;
    // (a call that is recorded into a graph has a workspace of its own; the default stream cannot be captured)
    if (need > 0 && stream && c10::hip::currentStreamCaptureStatusMayInitCtx() != c10::hip::CaptureStatus::None) Py_RETURN_NONE;

    const at::Tensor o = fresh(q.sizes(), out_dtype, q.device());
    const at::Tensor to = t[3] ? fresh(q.sizes(), out_dtype, q.device()) : at::Tensor();
    const at::Tensor lse = fresh({B, H, Lq}, at::kFloat, q.device());
    attn_jvp_opts opts = {};
    opts.in_dtype = f32 ? ATTN_JVP_FP32 : ATTN_JVP_BF16;
    opts.out_dtype = out_dtype == at::kFloat ? ATTN_JVP_OUT_FP32 : ATTN_JVP_OUT_INPUT;
    opts.stream = stream;
    opts.kernel = (int)kernel;
    opts.flags = (int)flags;
    opts.layout = (int)layout;
    Workspace ws;
    if (need > 0) {
        if (!ws.take(a[0], stream, need)) return nullptr;
        opts.workspace = ws.get().data_ptr();
        opts.workspace_bytes = (size_t)ws.get().numel();
    }
    const void* in[6];
    for (int i = 0; i < 6; ++i) in[i] = t[i] ? t[i]->data_ptr() : nullptr;
    void *po = o.data_ptr(), *pto = t[3] ? to.data_ptr() : nullptr;
    float* plse = static_cast<float*>(lse.data_ptr());
    const float scale = (float)PyFloat_AS_DOUBLE(a[6]);
    int rc;
    Py_BEGIN_ALLOW_THREADS      // (the tensors are held by the caller's arguments, the workspace by `ws`)
    rc = fwd_ex(in[0], in[1], in[2], in[3], in[4], in[5], po, pto, plse, (int)B, (int)H, (int)Lq, (int)Lkv, (int)d, scale, &opts);
    Py_END_ALLOW_THREADS
    if (rc != ATTN_JVP_OK) return PyLong_FromLong(rc);
    PyObject* out = PyTuple_New(3);
    if (!out) return nullptr;
    PyTuple_SET_ITEM(out, 0, THPVariable_Wrap(o));
    PyTuple_SET_ITEM(out, 1, t[3] ? THPVariable_Wrap(to) : Py_NewRef(Py_None));
    PyTuple_SET_ITEM(out, 2, THPVariable_Wrap(lse));
    return out;
    END_HANDLE_TH_ERRORS
}

// rmsnorm(x, tx, w, eps) -> (y, ty), an error code, or None
PyObject* rmsnorm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 4 || !rmsnorm_fwd || !plain_mode() || !PyFloat_CheckExact(a[3])) Py_RETURN_NONE;
    const at::Tensor *x = plain_tensor(a[0]), *tx = plain_tensor(a[1]), *w = plain_tensor(a[2]);
    if (!x || !tx || !w || x->dim() == 0) Py_RETURN_NONE;
    const auto dtype = x->scalar_type();
    const int64_t d = x->size(-1);
    if ((dtype != at::kFloat && dtype != at::kBFloat16) || tx->scalar_type() != dtype || tx->sizes() != x->sizes() || w->scalar_type() != at::kFloat ||
        w->dim() != 1 || w->size(0) != d || d <= 0 || !fits_int(d)) Py_RETURN_NONE;
    const auto index = x->device().index();
    if (c10::hip::current_device() != index || tx->device() != x->device() || w->device() != x->device()) Py_RETURN_NONE;
    const at::Tensor y = fresh(x->sizes(), dtype, x->device()), ty = fresh(x->sizes(), dtype, x->device());
    const hipStream_t stream = c10::hip::getCurrentHIPStream(index).stream();
    const void *px = x->data_ptr(), *ptx = tx->data_ptr();
    const float* pw = static_cast<const float*>(w->data_ptr());
    void *py = y.data_ptr(), *pty = ty.data_ptr();
    const long long rows = x->numel() / d;
    const float eps = (float)PyFloat_AS_DOUBLE(a[3]);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = rmsnorm_fwd(px, ptx, pw, py, pty, rows, (int)d, eps, dtype == at::kFloat ? ATTN_JVP_FP32 : ATTN_JVP_BF16, stream);
    Py_END_ALLOW_THREADS
    if (rc != ATTN_JVP_OK) return PyLong_FromLong(rc);
    PyObject* out = PyTuple_New(2);
    if (!out) return nullptr;
    PyTuple_SET_ITEM(out, 0, THPVariable_Wrap(y));
    PyTuple_SET_ITEM(out, 1, THPVariable_Wrap(ty));
    return out;
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"init", init, METH_VARARGS, nullptr},
    {"attn", (PyCFunction)(void*)attn, METH_FASTCALL, nullptr},
    {"rmsnorm", (PyCFunction)(void*)rmsnorm, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fast_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fast_call() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", BUILT_FOR_TORCH) != 0) Py_CLEAR(m);      // (binding.py compares it)
    return m;
}
