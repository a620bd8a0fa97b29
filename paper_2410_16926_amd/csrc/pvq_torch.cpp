// Native half of binding.py: takes torch tensors apart, allocates results and calls libpvq on the current
// stream.  What a call of a small matrix costs is host time (a kernel of 4 us behind 10 us of attribute
// lookups, ctypes conversions and 3 us for the stream object in Python; about 4 us from here, most of it the
// launch itself), so the whole way from the Python call to the C ABI is native.  Argument marshalling only.
//
// Every function returns its result, or the library's negative status as an int (binding.py raises PvqError
// from it).  The interpreter lock is released around the library call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "pvq.h"

namespace {

// raised as the named Python exception
struct bad_argument {
    PyObject *type;
    const char *text;
};

void *context(PyObject *o)
{
    if (o == Py_None) return nullptr;
    void *p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw bad_argument{nullptr, nullptr};
    return p;
}

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) throw bad_argument{PyExc_TypeError, "a torch tensor is wanted"};
    return THPVariable_Unpack(o);
}

void *data(const at::Tensor &t) { return t.unsafeGetTensorImpl()->mutable_data(); }

// the address of a tensor's data; None gives a null pointer
void *data_or_null(PyObject *o) { return o == Py_None ? nullptr : data(tensor(o)); }

int64_t number(PyObject *o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw bad_argument{nullptr, nullptr};
    return v;
}

int dtype_code(at::ScalarType t)
{
    switch (t) {
    case at::kFloat: return PVQ_F32;
    case at::kHalf: return PVQ_F16;
    case at::kBFloat16: return PVQ_BF16;
    default: throw bad_argument{PyExc_KeyError, "a dtype of float32, float16 or bfloat16 is wanted"};
    }
}

// a dtype argument, or `otherwise` for None
at::ScalarType scalar_type(PyObject *o, at::ScalarType otherwise)
{
    if (o == Py_None) return otherwise;
    if (!THPDtype_Check(o)) throw bad_argument{PyExc_TypeError, "a torch dtype is wanted"};
    return reinterpret_cast<THPDtype *>(o)->scalar_type;
}

at::Tensor new_tensor(at::IntArrayRef shape, at::ScalarType type, const at::Tensor &like)
{
    return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}

// rows, columns and row stride of a matrix with unit column stride; a single row is as long as it is wide
struct matrix_shape {
    int64_t rows, cols, ld;
};
matrix_shape matrix(const at::Tensor &t)
{
    if (t.dim() != 2) throw bad_argument{PyExc_ValueError, "a matrix is wanted"};
    return {t.size(0), t.size(1), t.size(0) > 1 ? t.stride(0) : std::max<int64_t>(t.size(1), 1)};
}

void *current_stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

struct without_lock {
    PyThreadState *state = PyEval_SaveThread();
    ~without_lock() { PyEval_RestoreThread(state); }
};

PyObject *status_or(int status, const at::Tensor &result)
{
    return status ? PyLong_FromLong(status) : THPVariable_Wrap(result);
}

// ---- packed planes -----------------------------------------------------------------------------------

struct planes {
    at::Tensor index, scale, rownorm;
};

// the planes of rows x cols for a context, or a negative status
int new_planes(const pvq_ctx *c, int64_t rows, int64_t cols, const at::Tensor &like, planes &p)
{
    size_t index_bytes = 0, scale_bytes = 0;
    int D = 0, scale_bits = 0;
    int status = pvq_packed_sizes(c, rows, cols, &index_bytes, &scale_bytes, nullptr);
    if (!status) status = pvq_ctx_info(c, &D, nullptr, nullptr, &scale_bits);
    if (status) return status;
    const int64_t n = std::max<int64_t>(rows, 1);
    p.index = new_tensor({rows, (int64_t)index_bytes / 4 / n}, at::kInt, like);
    p.scale = scale_bits ? new_tensor({rows, (int64_t)scale_bytes / 4 / n}, at::kInt, like)
                         : new_tensor({rows, cols / D}, at::kFloat, like);
    p.rownorm = new_tensor({rows}, at::kFloat, like);
    return PVQ_OK;
}

PyObject *wrap(const planes &p)
{
    PyObject *index = THPVariable_Wrap(p.index), *scale = THPVariable_Wrap(p.scale), *rownorm = THPVariable_Wrap(p.rownorm);
    PyObject *r = index && scale && rownorm ? PyTuple_Pack(3, index, scale, rownorm) : nullptr;
    Py_XDECREF(index); Py_XDECREF(scale); Py_XDECREF(rownorm);
    return r;
}

// ---- the calls ---------------------------------------------------------------------------------------

// (ctx, W, index, scale, rownorm, pulses): planes given, or None for new ones.  Returns None where the planes were
// given, else the three new ones.
PyObject *encode(PyObject *const *a)
{
    const pvq_ctx *c = (const pvq_ctx *)context(a[0]);
    const at::Tensor &W = tensor(a[1]);
    const matrix_shape m = matrix(W);
    const int dtype = dtype_code(W.scalar_type());
    const bool given = a[2] != Py_None;
    planes p;
    if (!given)
        if (const int status = new_planes(c, m.rows, m.cols, W, p)) return PyLong_FromLong(status);
    void *index = given ? data(tensor(a[2])) : data(p.index), *scale = given ? data_or_null(a[3]) : data(p.scale);
    void *rownorm = given ? data_or_null(a[4]) : data(p.rownorm), *pulses = data_or_null(a[5]);
    void *w = data(W), *stream = current_stream();
    int status;
    {
        without_lock unlocked;
        status = pvq_encode(c, w, dtype, m.rows, m.cols, m.ld, (uint32_t *)index, scale, (float *)rownorm, (int8_t *)pulses, stream);
    }
    if (status) return PyLong_FromLong(status);
    if (given) Py_RETURN_NONE;
    return wrap(p);
}

// (ctx, X, block, signs, index, scale, rownorm)
PyObject *rotate_encode(PyObject *const *a)
{
    const pvq_ctx *c = (const pvq_ctx *)context(a[0]);
    const at::Tensor &X = tensor(a[1]);
    const matrix_shape m = matrix(X);
    const int dtype = dtype_code(X.scalar_type()), block = (int)number(a[2]);
    const bool given = a[4] != Py_None;
    planes p;
    if (!given)
        if (const int status = new_planes(c, m.rows, m.cols, X, p)) return PyLong_FromLong(status);
    void *index = given ? data(tensor(a[4])) : data(p.index), *scale = given ? data_or_null(a[5]) : data(p.scale);
    void *rownorm = given ? data_or_null(a[6]) : data(p.rownorm);
    void *x = data(X), *signs = data_or_null(a[3]), *stream = current_stream();
    int status;
    {
        without_lock unlocked;
        status = pvq_rotate_encode(c, x, dtype, m.rows, m.cols, m.ld, block, (const uint8_t *)signs, (uint32_t *)index, scale, (float *)rownorm, stream);
    }
    if (status) return PyLong_FromLong(status);
    if (given) Py_RETURN_NONE;
    return wrap(p);
}

// (ctx, index, scale, rownorm, rows, cols, out_dtype or None, out or None)
PyObject *decode(PyObject *const *a)
{
    const pvq_ctx *c = (const pvq_ctx *)context(a[0]);
    const at::Tensor &index = tensor(a[1]);
    const int64_t rows = number(a[4]), cols = number(a[5]);
    const at::Tensor out = a[7] != Py_None ? tensor(a[7]) : new_tensor({rows, cols}, scalar_type(a[6], at::kFloat), index);
    const int dtype = dtype_code(out.scalar_type());
    const int64_t ld = rows > 1 ? out.stride(0) : std::max<int64_t>(cols, 1);
    void *i = data(index), *scale = data_or_null(a[2]), *rownorm = data_or_null(a[3]), *o = data(out), *stream = current_stream();
    int status;
    {
        without_lock unlocked;
        status = pvq_decode(c, (const uint32_t *)i, scale, (const float *)rownorm, rows, cols, o, dtype, ld, stream);
    }
    return status_or(status, out);
}

// (ctx, index, scale, rownorm, rows, cols, x, out or None)
PyObject *decode_gemv(PyObject *const *a)
{
    const pvq_ctx *c = (const pvq_ctx *)context(a[0]);
    const at::Tensor &index = tensor(a[1]), &x = tensor(a[6]);
    const int64_t rows = number(a[4]), cols = number(a[5]);
    if (x.dim() != 2 || x.scalar_type() != at::kBFloat16 || x.size(1) != cols)
        throw bad_argument{PyExc_AssertionError, "x is bfloat16 [batch][cols]"};
    const int64_t batch = x.size(0);
    const at::Tensor out = a[7] != Py_None ? tensor(a[7]) : new_tensor({batch, rows}, at::kFloat, x);
    const int64_t ldx = batch > 1 ? x.stride(0) : std::max<int64_t>(cols, 1), ldy = batch > 1 ? out.stride(0) : std::max<int64_t>(rows, 1);
    void *i = data(index), *scale = data_or_null(a[2]), *rownorm = data_or_null(a[3]), *xp = data(x), *o = data(out), *stream = current_stream();
    int status;
    {
        without_lock unlocked;
        status = pvq_decode_gemv(c, (const uint32_t *)i, scale, (const float *)rownorm, rows, cols, xp, (int)batch, ldx, (float *)o, ldy, stream);
    }
    return status_or(status, out);
}

// (X, block, signs, inverse, out or None, out_dtype or None)
PyObject *hadamard(PyObject *const *a)
{
    const at::Tensor &X = tensor(a[0]);
    if (X.dim() != 2) throw bad_argument{PyExc_ValueError, "a matrix is wanted"};
    const int64_t rows = X.size(0), cols = X.size(1);
    const at::Tensor out = a[4] != Py_None ? tensor(a[4]) : new_tensor({rows, cols}, scalar_type(a[5], X.scalar_type()), X);
    const int in_dtype = dtype_code(X.scalar_type()), out_dtype = dtype_code(out.scalar_type()), block = (int)number(a[1]);
    const int inverse = PyObject_IsTrue(a[3]);
    if (inverse < 0) throw bad_argument{nullptr, nullptr};
    const int64_t ldx = rows > 1 ? X.stride(0) : cols, ldy = rows > 1 ? out.stride(0) : cols;
    void *x = data(X), *signs = data_or_null(a[2]), *o = data(out), *stream = current_stream();
    int status;
    {
        without_lock unlocked;
        status = pvq_hadamard(x, in_dtype, rows, cols, ldx, block, (const uint8_t *)signs, inverse, o, out_dtype, ldy, stream);
    }
    return status_or(status, out);
}

// (): the current stream's handle
PyObject *stream(PyObject *const *) { return PyLong_FromVoidPtr(current_stream()); }

// ---- the module --------------------------------------------------------------------------------------

template <PyObject *(*F)(PyObject *const *), int N>
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    try {
        if (n != N) throw bad_argument{PyExc_TypeError, "wrong number of arguments"};
        return F(args);
    } catch (const bad_argument &e) {
        if (e.type) PyErr_SetString(e.type, e.text);        // (else the interpreter has its error already)
    } catch (...) {
        torch::translate_exception_to_python(std::current_exception());
    }
    return nullptr;
}

#define PVQ_METHOD(NAME, N) {#NAME, (PyCFunction)(void (*)(void))call<NAME, N>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {PVQ_METHOD(encode, 6), PVQ_METHOD(rotate_encode, 7), PVQ_METHOD(decode, 8), PVQ_METHOD(decode_gemv, 8),
                         PVQ_METHOD(hadamard, 6), PVQ_METHOD(stream, 0), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pvq_torch", "libpvq's calls on torch tensors", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// What the module was built for, for build.py, which looks for this text in the file before the module is loaded.
extern "C" __attribute__((used, visibility("default"))) const char pvq_torch_built_for[] = PVQ_BUILT_FOR;

PyMODINIT_FUNC PyInit__pvq_torch(void) { return PyModule_Create(&module); }
