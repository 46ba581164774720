// The Python side of a call, natively: what binding.py has in hand (a descriptor array that it made earlier, tensors, small
// integers) becomes the arguments of a C function of libtmask.so, whose address binding.py passes.  A call of one small kernel
// is bound by its host time, and half of that was the reading of tensor attributes and the conversion of arguments one by one
// (one 256 x 64 layer 5.1 -> 4.5 us back to back, a product with 16 tokens 5.8 -> 3.5).
//
// Every function returns the C function's result, or None where something is not as it usually is (a type, a shape, a value
// outside int, a tensor that has no memory of its own or none on the device): binding.py then goes through the same arguments step by step and raises
// what is to be raised.  No function raises by itself, and none keeps anything between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstdint>
#include <type_traits>

#include "../../include/tmask.h"

#ifndef TMASK_BUILT_FOR
#error "the build names the torch and the Python that the module is for"
#endif

namespace {

// The C functions come as addresses; their types are those of the header, or this does not compile.
template <typename Desc>
using batch_fn = int(const Desc *, int, tmask_dtype, int, int, tmask_mask_fmt, void *, size_t, void *);
static_assert(std::is_same_v<decltype(tmask_approx), batch_fn<tmask_mat>> && std::is_same_v<decltype(tmask_exact), batch_fn<tmask_mat>> &&
              std::is_same_v<decltype(tmask_prune_1d), batch_fn<tmask_mat>> && std::is_same_v<decltype(tmask_apply_pack), batch_fn<tmask_pack_desc>> &&
              std::is_same_v<decltype(tmask_approx_pack), batch_fn<tmask_fused_desc>>, "the functions that batch() is called with");

bool as_int(PyObject *o, int *out)
{
    if (!PyLong_Check(o))
        return false;
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow || v < INT_MIN || v > INT_MAX)
        return false;
    *out = (int)v;
    return true;
}

bool as_int64(PyObject *o, int64_t *out)
{
    if (!PyLong_Check(o))
        return false;
    int overflow = 0;
    *out = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}

bool as_address(PyObject *o, void **out)
{
    if (!PyLong_Check(o))
        return false;
    *out = PyLong_AsVoidPtr(o);
    return !PyErr_Occurred() && *out;
}

bool as_tensor(PyObject *o, const at::Tensor **out)
{
    if (!THPVariable_CheckExact(o))          // subclasses have their own ideas about attributes
        return false;
    *out = &THPVariable_Unpack(o);
    return true;
}

// the current stream's handle if None, else that of a torch stream
bool as_stream(PyObject *o, void **out)
{
    if (o == Py_None) {
        *out = (void *)c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    PyObject *const handle = PyObject_GetAttrString(o, "cuda_stream");
    bool ok = handle && PyLong_Check(handle);
    if (ok) {
        *out = PyLong_AsVoidPtr(handle);         // the default stream's is 0
        ok = !PyErr_Occurred();
    }
    Py_XDECREF(handle);
    if (!ok)
        PyErr_Clear();
    return ok;
}

bool as_workspace(PyObject *o, void **out, size_t *bytes)
{
    *out = nullptr;
    *bytes = 0;
    if (o == Py_None)
        return true;
    const at::Tensor *t;
    if (!as_tensor(o, &t) || !t->is_cuda())
        return false;
    *out = t->data_ptr();
    *bytes = (size_t)t->numel() * (size_t)t->element_size();
    return true;
}

// function, descriptor array, n, dtype, N, M, mask format: the arguments that most calls begin with
struct Head {
    void *fn, *descs;
    int n, dt, N, M, fmt;
};

bool as_head(PyObject *const *a, Head *h)
{
    return as_address(a[0], &h->fn) && as_address(a[1], &h->descs) && as_int(a[2], &h->n) && as_int(a[3], &h->dt) && as_int(a[4], &h->N) &&
           as_int(a[5], &h->M) && as_int(a[6], &h->fmt);
}

// The arguments of a call are gathered by `gather`, which returns whether they are the usual ones, and the call is made without
// the interpreter's lock, as ctypes makes it.
template <typename Gather, typename Call>
PyObject *run(Gather gather, Call call)
{
    bool usual = false;
    try {
        usual = gather();
    } catch (...) {
        usual = false;
    }
    if (PyErr_Occurred())
        PyErr_Clear();
    if (!usual)
        Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// batch(function, descs, n, dtype, N, M, mask format, workspace, stream)
PyObject *batch(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 9)
        Py_RETURN_NONE;
    Head h;
    void *ws, *stream;
    size_t bytes;
    return run([&] { return as_head(a, &h) && as_workspace(a[7], &ws, &bytes) && as_stream(a[8], &stream); },
               [&] {
                   return ((batch_fn<void> *)h.fn)(h.descs, h.n, (tmask_dtype)h.dt, h.N, h.M, (tmask_mask_fmt)h.fmt, ws, bytes, stream);
               });
}

// dense(function, descs, n, dtype, N, M, mask format, stream)
PyObject *dense(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 8)
        Py_RETURN_NONE;
    Head h;
    void *stream;
    return run([&] { return as_head(a, &h) && as_stream(a[7], &stream); },
               [&] {
                   return ((decltype(&tmask_approx_dense))h.fn)((const tmask_mask_dense_desc *)h.descs, h.n, (tmask_dtype)h.dt, h.N, h.M,
                                                                (tmask_mask_fmt)h.fmt, stream);
               });
}

// score(function, descs, n, dtype, N, M, mask format, out, bytes of out at least, per_block, workspace, stream)
PyObject *score(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 12)
        Py_RETURN_NONE;
    Head h;
    void *out, *per_block = nullptr, *ws, *stream;
    size_t bytes;
    return run(
        [&] {
            const at::Tensor *o, *p;
            int64_t least;
            if (!as_head(a, &h) || !as_tensor(a[7], &o) || !as_int64(a[8], &least))
                return false;
            if (o->numel() * o->element_size() < least || !o->is_cuda() || !o->is_contiguous())
                return false;
            out = o->data_ptr();
            if (a[9] != Py_None) {
                if (!as_tensor(a[9], &p) || p->scalar_type() != at::kFloat || !p->is_cuda() || !p->is_contiguous())
                    return false;
                per_block = p->data_ptr();
            }
            return as_workspace(a[10], &ws, &bytes) && as_stream(a[11], &stream);
        },
        [&] {
            return ((decltype(&tmask_score))h.fn)((const tmask_mat *)h.descs, h.n, (tmask_dtype)h.dt, h.N, h.M, (tmask_mask_fmt)h.fmt,
                                                  (tmask_score_out *)out, (float *)per_block, ws, bytes, stream);
        });
}

// spmm24(function, vals, idx, rows, cols, x, y, stream)
PyObject *spmm24(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 8)
        Py_RETURN_NONE;
    const at::Tensor *vals, *idx, *x, *y;
    int64_t rows, cols;
    void *fn, *pv, *pi, *px, *py, *stream;
    int64_t ld_x, ld_y, tokens;
    int dt;
    return run(
        [&] {
            if (!as_address(a[0], &fn) || !as_tensor(a[1], &vals) || !as_tensor(a[2], &idx) || !as_int64(a[3], &rows) || !as_int64(a[4], &cols) ||
                !as_tensor(a[5], &x) || !as_tensor(a[6], &y))
                return false;
            if (x->scalar_type() != at::kBFloat16 || vals->scalar_type() != at::kBFloat16 || idx->scalar_type() != at::kByte)
                return false;
            if (y->scalar_type() != at::kFloat && y->scalar_type() != at::kBFloat16)
                return false;
            if (x->dim() != 2 || y->dim() != 2 || vals->dim() != 2 || idx->dim() != 2 || x->stride(1) != 1 || y->stride(1) != 1 ||
                !x->is_cuda() || !y->is_cuda() || !vals->is_cuda() || !idx->is_cuda() || !vals->is_contiguous() || !idx->is_contiguous())
                return false;
            if (cols < 0 || x->size(1) != cols || y->size(0) != x->size(0) || y->size(1) != rows || vals->size(0) != rows ||
                vals->size(1) != cols / 2 || idx->size(0) != rows || idx->size(1) != cols / 8)
                return false;
            pv = vals->data_ptr(); pi = idx->data_ptr(); px = x->data_ptr(); py = y->data_ptr();
            ld_x = x->stride(0); ld_y = y->stride(0); tokens = x->size(0);
            dt = y->scalar_type() == at::kFloat ? 0 : 1;
            return as_stream(a[7], &stream);
        },
        [&] {
            return ((decltype(&tmask_spmm24))fn)(pv, pi, rows, cols, px, ld_x, py, ld_y, tokens, (tmask_dtype)dt, stream);
        });
}

PyMethodDef kMethods[] = {{"batch", (PyCFunction)(void (*)(void))batch, METH_FASTCALL, nullptr},
                          {"dense", (PyCFunction)(void (*)(void))dense, METH_FASTCALL, nullptr},
                          {"score", (PyCFunction)(void (*)(void))score, METH_FASTCALL, nullptr},
                          {"spmm24", (PyCFunction)(void (*)(void))spmm24, METH_FASTCALL, nullptr},
                          {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_calls", nullptr, 0, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void)
{
    PyObject *const m = PyModule_Create(&kModule);
    if (m && PyModule_AddStringConstant(m, "built_for", TMASK_BUILT_FOR) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
