// The common calls of the Python binding, from torch tensors straight to the C ABI.
//
// A small product is bound by its host path: the kernel of a 4096-row SpMM takes 4.6 us, its launch 3 us, and marshalling
// one call in Python 3 us (attention, with more operands, a second launch and a workspace: 7 us).  Here the checks, the
// allocation of the result and of the workspace and the call are compiled; what is left for Python is to pass the
// tensors.  Every function takes (address of the fs_format, tensors, ..., stream handle; before it, where a workspace may be
// needed, the stream object or None for the current stream) and returns the result tensor,
// the library's status as an int where the call failed, or None where an argument is not what the call expects, which
// the binding's checks in Python then name.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/StreamGuard.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/Stream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "flashsparse.h"

namespace {

// The library's entry points, from the shared object the binding has loaded (see bind).
struct Entry {
    decltype(&fs_spmm_workspace_bytes) spmm_work;
    decltype(&fs_attention_workspace_bytes) attention_work;
    decltype(&fs_edge_softmax_workspace_bytes) softmax_work;
    decltype(&fs_spmm) spmm;
    decltype(&fs_sddmm) sddmm;
    decltype(&fs_attention) attention;
    decltype(&fs_sddmm_spmm) sddmm_spmm;
    decltype(&fs_edge_softmax) softmax;
    decltype(&fs_edge_softmax_backward) softmax_backward;
    decltype(&fs_csr_to_blk) csr_to_blk;
    decltype(&fs_blk_to_csr) blk_to_csr;
    decltype(&fs_gather16) gather16;
} g;
constexpr Py_ssize_t kEntries = sizeof(Entry) / sizeof(void *);

const fs_format *format_at(PyObject *o) { return (const fs_format *)PyLong_AsVoidPtr(o); }
void *pointer(PyObject *o) { return PyLong_AsVoidPtr(o); }

bool of_format(const at::Tensor &t, const fs_format *f)
{
    return t.is_cuda() && t.scalar_type() == (f->dtype == FS_F16 ? at::kHalf : at::kBFloat16);
}
bool matrix(PyObject *o, const fs_format *f, int64_t rows)
{
    if (!THPVariable_Check(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.dim() == 2 && of_format(t, f) && t.stride(1) == 1 && t.size(0) == rows;
}
bool flat(PyObject *o, const fs_format *f, int64_t numel)
{
    if (!THPVariable_Check(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    return of_format(t, f) && t.is_contiguous() && t.numel() == numel;
}

PyObject *finish(const at::Tensor &out, fs_status st)
{
    return st == FS_OK ? THPVariable_Wrap(out) : PyLong_FromLong((long)st);
}

bool stream_or_none(PyObject *o) { return o == Py_None || THPStream_Check(o); }

// A buffer that is given back when the call returns, from the memory of the stream `on` that the kernels run on (None: the
// current one): only work on that stream may have it next.
at::Tensor temporary_on(const at::Tensor &like, int64_t bytes, PyObject *on)
{
    c10::OptionalStreamGuard guard;
    if (on != Py_None) {
        const THPStream *s = (const THPStream *)on;
        guard.reset_stream(c10::Stream::unpack3(s->stream_id, (c10::DeviceIndex)s->device_index, (c10::DeviceType)s->device_type));
    }
    return at::empty({bytes}, like.options().dtype(at::kByte));
}

// A workspace holds the parts of cut windows: without any there is none.
struct Work {
    at::Tensor t;
    void *p = nullptr;
    size_t bytes = 0;
    fs_status st = FS_OK;
    template <typename Query>
    Work(const fs_format *f, const at::Tensor &like, PyObject *on, Query query)
    {
        if (f->n_split_items == 0) return;
        st = query(&bytes);
        if (st != FS_OK || bytes == 0) return;
        t = temporary_on(like, (int64_t)bytes, on);
        p = t.data_ptr();
    }
};

// The C call without the interpreter's lock: a launch may have to wait for room in the queue.
#define FS_CALL(st, call)      \
    Py_BEGIN_ALLOW_THREADS     \
    st = call;                 \
    Py_END_ALLOW_THREADS

PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != kEntries) { PyErr_SetString(PyExc_TypeError, "wrong number of entry points"); return nullptr; }
    void **to = (void **)&g;
    for (Py_ssize_t i = 0; i < n; i++) to[i] = pointer(a[i]);
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

#define FS_ENTRY(name, args)                                                                             \
    PyObject *name(PyObject *, PyObject *const *a, Py_ssize_t n)                                         \
    {                                                                                                    \
        HANDLE_TH_ERRORS                                                                                 \
        if (n != args) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; } \
        const fs_format *f = format_at(a[0]);                                                            \
        void *stream = pointer(a[args - 1]);                                                             \
        if (PyErr_Occurred()) return nullptr;                                                            \
        fs_status st = FS_OK;
#define FS_ENTRY_END     \
        END_HANDLE_TH_ERRORS \
    }

FS_ENTRY(spmm, 5)  // format, B, values or None, stream object, stream
    if (!matrix(a[1], f, f->K) || !(a[2] == Py_None || flat(a[2], f, f->V * f->nvec)) || !stream_or_none(a[3])) Py_RETURN_NONE;
    const at::Tensor &B = THPVariable_Unpack(a[1]);
    const int64_t N = B.size(1);
    const void *vals = a[2] == Py_None ? nullptr : THPVariable_Unpack(a[2]).data_ptr();
    at::Tensor out = at::empty({f->M, N}, B.options());
    Work w(f, B, a[3], [&](size_t *b) { return g.spmm_work(f, N, b); });
    if (w.st != FS_OK) return finish(out, w.st);
    FS_CALL(st, g.spmm(f, vals, B.data_ptr(), N, B.stride(0), out.data_ptr(), N, w.p, w.bytes, stream))
    return finish(out, st);
FS_ENTRY_END

FS_ENTRY(sddmm, 5)  // format, X, Y, true: vals_blk layout, false: CSR order, stream
    if (!matrix(a[1], f, f->M) || !matrix(a[2], f, f->K)) Py_RETURN_NONE;
    const at::Tensor &X = THPVariable_Unpack(a[1]), &Y = THPVariable_Unpack(a[2]);
    const int64_t d = X.size(1);
    if (Y.size(1) != d) Py_RETURN_NONE;
    const bool blocked = a[3] == Py_True;
    at::Tensor out = at::empty({blocked ? f->V * f->nvec : f->nnz}, X.options());
    FS_CALL(st, g.sddmm(f, X.data_ptr(), X.stride(0), Y.data_ptr(), Y.stride(0), d, blocked ? out.data_ptr() : nullptr,
                        blocked ? nullptr : out.data_ptr(), stream))
    return finish(out, st);
FS_ENTRY_END

FS_ENTRY(attention, 8)  // format, X, Y, H, scale, true: with the softmax, stream object, stream
    if (!matrix(a[1], f, f->M) || !matrix(a[2], f, f->K) || !matrix(a[3], f, f->K) || !stream_or_none(a[6])) Py_RETURN_NONE;
    const at::Tensor &X = THPVariable_Unpack(a[1]), &Y = THPVariable_Unpack(a[2]), &H = THPVariable_Unpack(a[3]);
    const int64_t d = X.size(1), N = H.size(1);
    if (Y.size(1) != d) Py_RETURN_NONE;
    const float scale = (float)PyFloat_AsDouble(a[4]);
    if (PyErr_Occurred()) return nullptr;
    at::Tensor out = at::empty({f->M, N}, H.options());
    Work w(f, H, a[6], [&](size_t *b) { return g.attention_work(f, N, b); });
    if (w.st != FS_OK) return finish(out, w.st);
    FS_CALL(st, (a[5] == Py_True ? g.attention : g.sddmm_spmm)(f, X.data_ptr(), X.stride(0), Y.data_ptr(), Y.stride(0), d, scale,
                                                               H.data_ptr(), N, H.stride(0), out.data_ptr(), N, w.p, w.bytes, stream))
    return finish(out, st);
FS_ENTRY_END

FS_ENTRY(softmax, 5)  // format, values, scale, stream object, stream
    if (!flat(a[1], f, f->V * f->nvec) || !stream_or_none(a[3])) Py_RETURN_NONE;
    const at::Tensor &v = THPVariable_Unpack(a[1]);
    const float scale = (float)PyFloat_AsDouble(a[2]);
    if (PyErr_Occurred()) return nullptr;
    at::Tensor out = at::empty(v.sizes(), v.options());
    Work w(f, v, a[3], [&](size_t *b) { return g.softmax_work(f, b); });
    if (w.st != FS_OK) return finish(out, w.st);
    FS_CALL(st, g.softmax(f, v.data_ptr(), out.data_ptr(), scale, w.p, w.bytes, stream))
    return finish(out, st);
FS_ENTRY_END

FS_ENTRY(softmax_backward, 6)  // format, probabilities, their gradient, scale, stream object, stream
    if (!flat(a[1], f, f->V * f->nvec) || !flat(a[2], f, f->V * f->nvec) || !stream_or_none(a[4])) Py_RETURN_NONE;
    const at::Tensor &p = THPVariable_Unpack(a[1]), &gr = THPVariable_Unpack(a[2]);
    const float scale = (float)PyFloat_AsDouble(a[3]);
    if (PyErr_Occurred()) return nullptr;
    at::Tensor out = at::empty(p.sizes(), p.options());
    Work w(f, p, a[4], [&](size_t *b) { return g.softmax_work(f, b); });
    if (w.st != FS_OK) return finish(out, w.st);
    FS_CALL(st, g.softmax_backward(f, p.data_ptr(), gr.data_ptr(), scale, out.data_ptr(), w.p, w.bytes, stream))
    return finish(out, st);
FS_ENTRY_END

FS_ENTRY(csr_to_blk, 3)  // format, values in CSR order, stream
    if (!flat(a[1], f, f->nnz)) Py_RETURN_NONE;
    const at::Tensor &v = THPVariable_Unpack(a[1]);
    at::Tensor out = at::empty({f->V * f->nvec}, v.options());
    FS_CALL(st, g.csr_to_blk(f, v.data_ptr(), out.data_ptr(), stream))
    return finish(out, st);
FS_ENTRY_END

FS_ENTRY(blk_to_csr, 3)  // format, values in vals_blk layout, stream
    if (!flat(a[1], f, f->V * f->nvec)) Py_RETURN_NONE;
    const at::Tensor &v = THPVariable_Unpack(a[1]);
    at::Tensor out = at::empty({f->nnz}, v.options());
    FS_CALL(st, g.blk_to_csr(f, v.data_ptr(), out.data_ptr(), stream))
    return finish(out, st);
FS_ENTRY_END

PyObject *gather16(PyObject *, PyObject *const *a, Py_ssize_t n)  // source, indices, stream
{
    HANDLE_TH_ERRORS
    if (n != 3) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }
    void *stream = pointer(a[2]);
    if (PyErr_Occurred()) return nullptr;
    if (!THPVariable_Check(a[0]) || !THPVariable_Check(a[1])) Py_RETURN_NONE;
    const at::Tensor &src = THPVariable_Unpack(a[0]), &idx = THPVariable_Unpack(a[1]);
    if (!src.is_cuda() || !idx.is_cuda() || idx.scalar_type() != at::kInt || src.element_size() != 2 || !src.is_contiguous() ||
        !idx.is_contiguous())
        Py_RETURN_NONE;
    at::Tensor out = at::empty({idx.numel()}, src.options());
    fs_status st;
    FS_CALL(st, g.gather16(src.data_ptr(), (const int32_t *)idx.data_ptr(), idx.numel(), out.data_ptr(), stream))
    return finish(out, st);
    END_HANDLE_TH_ERRORS
}

// What the calls made through ctypes need of the above.
PyObject *temporary(PyObject *, PyObject *const *a, Py_ssize_t n)  // bytes, a tensor on the device, stream object or None
{
    HANDLE_TH_ERRORS
    if (n != 3) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }
    const int64_t bytes = PyLong_AsLongLong(a[0]);
    if (PyErr_Occurred()) return nullptr;
    if (!THPVariable_Check(a[1]) || !stream_or_none(a[2])) Py_RETURN_NONE;
    return THPVariable_Wrap(temporary_on(THPVariable_Unpack(a[1]), bytes, a[2]));
    END_HANDLE_TH_ERRORS
}

PyObject *holds16(PyObject *, PyObject *const *a, Py_ssize_t n)  // a tensor; does it hold so many 16-bit elements, side by side on a GPU?
{
    HANDLE_TH_ERRORS
    if (n != 2) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }
    const int64_t numel = PyLong_AsLongLong(a[1]);
    if (PyErr_Occurred()) return nullptr;
    if (!THPVariable_Check(a[0])) Py_RETURN_FALSE;
    const at::Tensor &t = THPVariable_Unpack(a[0]);
    return PyBool_FromLong(t.is_cuda() && t.element_size() == 2 && t.is_contiguous() && t.numel() >= numel);
    END_HANDLE_TH_ERRORS
}

#define FS_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FS_METHOD(bind), FS_METHOD(spmm), FS_METHOD(sddmm), FS_METHOD(attention), FS_METHOD(softmax),
                         FS_METHOD(softmax_backward), FS_METHOD(csr_to_blk), FS_METHOD(blk_to_csr), FS_METHOD(gather16),
                         FS_METHOD(temporary), FS_METHOD(holds16),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fs_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fs_torch(void) { return PyModule_Create(&module); }
