// The calls of mxq.py in native code: argument checks, output allocation and the call into libmxq without
// an interpreter in between.  (Three allocations and a dozen arguments cost 11 us from Python, twice what a
// small call takes on the GPU.)  Nothing is decided here that mxq.py does not decide: every function either does
// what the Python form does or returns None BEFORE it has done anything, and then the Python form runs, raises
// its errors, or handles what is rarer (tensor subclasses, active modes, other number types).  A library status
// other than 0 comes back as an int.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/ops/empty.h>
#include <ATen/record_function.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "../../include/mxq.h"

namespace {

// libmxq's functions, handed over by mxq.py from the library that it has loaded.
decltype(&mxq_quantize) p_quantize;
decltype(&mxq_quantize_hier) p_quantize_hier;
decltype(&mxq_quantize_batch) p_quantize_batch;
decltype(&mxq_tensor_absmax) p_tensor_absmax;
decltype(&mxq_dequantize) p_dequantize;
decltype(&mxq_dequantize_hier) p_dequantize_hier;
decltype(&mxq_clip_sse) p_clip_sse;
decltype(&mxq_histogram) p_histogram;

// Modes see the Python form's calls of torch; here they would see only part of them.
bool modes_active() { return at::impl::torch_function_mode_enabled() || c10::impl::dispatch_mode_enabled(); }

// Keys of tensors that are not simply their storage (wrappers of transforms, lazy conjugates and negatives).
const c10::DispatchKeySet kNotPlain({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                     c10::DispatchKey::Functionalize, c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
                                     c10::DispatchKey::ZeroTensor});

// A plain contiguous strided tensor on the GPU, or null.
const at::Tensor* plain(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || t.key_set().has_any(kNotPlain) || !t.has_storage() ||
        !t.is_contiguous())
        return nullptr;
    return &t;
}

const at::Tensor* buffer(PyObject* o, int64_t bytes, at::ScalarType type)
{
    const at::Tensor* t = plain(o);
    return (t && t->scalar_type() == type && t->numel() * (int64_t)t->element_size() >= bytes) ? t : nullptr;
}

bool integer(PyObject* o, long lo, long hi, int* out)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || v < lo || v > hi) return false;
    *out = (int)v;
    return true;
}

// 2, 4 .. 128: any other block size is the Python form's to refuse.
bool block_size(PyObject* o, int* out) { return integer(o, 2, 128, out) && (*out & (*out - 1)) == 0; }

bool number(PyObject* o, float* out)
{
    if (!PyFloat_CheckExact(o)) return false;
    *out = (float)PyFloat_AS_DOUBLE(o);
    return true;
}

int dtype_code(const at::Tensor& t)
{
    return t.scalar_type() == at::kBFloat16 ? MXQ_DT_BF16 : t.scalar_type() == at::kFloat ? MXQ_DT_F32 : -1;
}

void* ptr(const at::Tensor& t) { return t.data_ptr(); }

void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

// Nothing has asked to see a new tensor made, or to fill it: a tracer or a transform adds its key to the thread's, a profiler
// its callbacks, deterministic mode has new memory filled.
bool nothing_watches()
{
    const c10::DispatchKeySet added = c10::impl::tls_local_dispatch_key_set().included_ - c10::default_included_set;
    return added.empty() && !at::globalContext().deterministicAlgorithms() && !at::hasCallbacks();
}

// New tensors of one call: what at::empty ends at for a GPU, without its two dispatches (0.70 -> 0.47 us, three of them in a
// small call of 6 us).  Whether something watches is asked once, at the first (asked for each of them, the callbacks too, a small
// call takes 1 to 1.5 % longer: three outputs of 16 x 4096 5.56 -> 5.71 us).
struct NewOutputs {
    int direct = -1;
    at::Tensor operator()(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like)
    {
        if (direct < 0) direct = nothing_watches();
        if (direct) return at::detail::empty_cuda(shape, type, like.device(), std::nullopt);
        return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
    }
};

PyObject* none() { Py_RETURN_NONE; }

struct Unlocked {                                            // as ctypes calls: without the interpreter's lock
    PyThreadState* s = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(s); }
};

// A 2-D input of whole blocks.
struct Input {
    const at::Tensor* x = nullptr;
    int64_t rows = 0, cols = 0, blocks = 0;
    int block = 0, dt = -1;
    bool set(PyObject* o, PyObject* b)
    {
        x = plain(o);
        if (!x || x->dim() != 2 || (dt = dtype_code(*x)) < 0 || !block_size(b, &block)) return false;
        rows = x->size(0);
        cols = x->size(1);
        if (cols % block != 0) return false;
        blocks = rows * (cols / block);
        return true;
    }
};

// Output triple: the caller's buffers or new ones.
struct Outputs {
    at::Tensor codes, scales, sse;
    bool check(const Input& in, PyObject* c, PyObject* s, PyObject* e) const
    {
        return (c == Py_None || buffer(c, in.rows * in.cols / 2, at::kByte)) && (s == Py_None || buffer(s, in.blocks, at::kByte)) &&
               (e == Py_None || buffer(e, 4 * in.blocks, at::kFloat));
    }
    void make(NewOutputs& new_empty, const Input& in, PyObject* c, PyObject* s, PyObject* e, bool want_sse)
    {
        codes = c != Py_None ? THPVariable_Unpack(c) : new_empty({in.rows, in.cols / 2}, at::kByte, *in.x);
        scales = s != Py_None ? THPVariable_Unpack(s) : new_empty({in.rows, in.cols / in.block}, at::kByte, *in.x);
        if (e != Py_None) sse = THPVariable_Unpack(e);
        else if (want_sse) sse = new_empty({in.rows, in.cols / in.block}, at::kFloat, *in.x);
    }
    float* sse_ptr() const { return sse.defined() ? (float*)ptr(sse) : nullptr; }
};

PyObject* wrapped(const at::Tensor& t)
{
    if (!t.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(t);
}

PyObject* tuple_of(std::initializer_list<at::Tensor> ts)
{
    PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
    if (!r) return nullptr;
    Py_ssize_t i = 0;
    for (const at::Tensor& t : ts) {
        PyObject* o = wrapped(t);
        if (!o) { Py_DECREF(r); return nullptr; }
        PyTuple_SET_ITEM(r, i++, o);
    }
    return r;
}

// quantize(x, block, scale_fmt, recipe, tensor_scale, codes, scales, sse, want_sse, elem_fmt)
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Input in;
    Outputs out;
    NewOutputs new_empty;
    int fmt, recipe, elem, want;
    float T;
    if (n != 10 || modes_active() || !in.set(a[0], a[1]) || !integer(a[2], 0, 255, &fmt) || !integer(a[3], 0, 255, &recipe) ||
        !number(a[4], &T) || !out.check(in, a[5], a[6], a[7]) || !integer(a[9], 0, 255, &elem))
        return none();
    want = PyObject_IsTrue(a[8]);
    if (want < 0) return nullptr;
    out.make(new_empty, in, a[5], a[6], a[7], want != 0);
    int status;
    {
        void* st = stream();
        Unlocked u;
        status = p_quantize(ptr(*in.x), in.rows, in.cols, in.block, elem, fmt, recipe, T, (uint8_t*)ptr(out.codes),
                            (uint8_t*)ptr(out.scales), out.sse_ptr(), in.dt, st);
    }
    if (status != MXQ_OK) return PyLong_FromLong(status);
    return tuple_of({out.codes, out.scales, out.sse});
    END_HANDLE_TH_ERRORS
}

// quantize_hier(x, block, scale_fmt, recipe, absmax, tensor_scale, codes, scales, sse, want_sse, elem_fmt)
PyObject* quantize_hier(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Input in;
    Outputs out;
    NewOutputs new_empty;
    int fmt, recipe, elem, want;
    if (n != 11 || modes_active() || !in.set(a[0], a[1]) || !integer(a[2], 0, 255, &fmt) || !integer(a[3], 0, 255, &recipe) ||
        !buffer(a[4], 4, at::kFloat) || !(a[5] == Py_None || buffer(a[5], 4, at::kFloat)) || !out.check(in, a[6], a[7], a[8]) ||
        !integer(a[10], 0, 255, &elem) || in.rows * in.cols == 0)
        return none();
    want = PyObject_IsTrue(a[9]);
    if (want < 0) return nullptr;
    const at::Tensor& absmax = THPVariable_Unpack(a[4]);
    const at::Tensor t = a[5] != Py_None ? THPVariable_Unpack(a[5]) : new_empty({1}, at::kFloat, *in.x);     // the kernel writes it
    out.make(new_empty, in, a[6], a[7], a[8], want != 0);
    int status;
    {
        void* st = stream();
        Unlocked u;
        status = p_quantize_hier(ptr(*in.x), in.rows, in.cols, in.block, elem, fmt, recipe, (const float*)ptr(absmax), (float*)ptr(t),
                                 (uint8_t*)ptr(out.codes), (uint8_t*)ptr(out.scales), out.sse_ptr(), in.dt, st);
    }
    if (status != MXQ_OK) return PyLong_FromLong(status);
    return tuple_of({out.codes, out.scales, out.sse, t});
    END_HANDLE_TH_ERRORS
}

// quantize_batch(list of x, block, scale_fmt, recipe, want_sse, elem_fmt), outputs allocated here
PyObject* quantize_batch(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int fmt, recipe, elem, want;
    if (n != 6 || modes_active() || !PyList_CheckExact(a[0]) || !integer(a[2], 0, 255, &fmt) || !integer(a[3], 0, 255, &recipe) ||
        !integer(a[5], 0, 255, &elem))
        return none();
    const Py_ssize_t count = PyList_GET_SIZE(a[0]);
    std::vector<Input> in((size_t)count);
    if (count == 0) return none();
    for (Py_ssize_t i = 0; i < count; ++i)
        if (!in[i].set(PyList_GET_ITEM(a[0], i), a[1]) || in[i].dt != in[0].dt) return none();
    want = PyObject_IsTrue(a[4]);
    if (want < 0) return nullptr;
    std::vector<Outputs> out((size_t)count);
    NewOutputs new_empty;
    std::vector<mxq_tensor> t((size_t)count);
    for (Py_ssize_t i = 0; i < count; ++i) {
        out[i].make(new_empty, in[i], Py_None, Py_None, Py_None, want != 0);
        t[i] = mxq_tensor{ptr(*in[i].x), in[i].rows, in[i].cols, (uint8_t*)ptr(out[i].codes), (uint8_t*)ptr(out[i].scales), out[i].sse_ptr()};
    }
    int status;
    {
        void* st = stream();
        Unlocked u;
        status = p_quantize_batch(t.data(), (int)count, in[0].block, elem, fmt, recipe, in[0].dt, st);
    }
    if (status != MXQ_OK) return PyLong_FromLong(status);
    PyObject* r = PyList_New(count);
    if (!r) return nullptr;
    for (Py_ssize_t i = 0; i < count; ++i) {
        PyObject* o = tuple_of({out[i].codes, out[i].scales, out[i].sse});
        if (!o) { Py_DECREF(r); return nullptr; }
        PyList_SET_ITEM(r, i, o);
    }
    return r;
    END_HANDLE_TH_ERRORS
}

// tensor_absmax(x, out)
PyObject* tensor_absmax(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor* x = (n == 2 && !modes_active()) ? plain(a[0]) : nullptr;
    if (!x || dtype_code(*x) < 0 || !(a[1] == Py_None || buffer(a[1], 4, at::kFloat))) return none();
    const at::Tensor out = a[1] != Py_None ? THPVariable_Unpack(a[1]) : NewOutputs()({1}, at::kFloat, *x);
    const int64_t rows = x->dim() == 2 ? x->size(0) : 1, cols = x->dim() == 2 ? x->size(1) : x->numel();
    int status;
    {
        void* st = stream();
        Unlocked u;
        status = p_tensor_absmax(ptr(*x), rows, cols, dtype_code(*x), (float*)ptr(out), st);
    }
    return status != MXQ_OK ? PyLong_FromLong(status) : wrapped(out);
    END_HANDLE_TH_ERRORS
}

// dequantize(codes, scales, block, scale_fmt, tensor_scale, out_dtype, out, elem_fmt)
PyObject* dequantize(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int block, fmt, elem;
    const at::Tensor* codes = (n == 8 && !modes_active()) ? plain(a[0]) : nullptr;
    if (!codes || codes->dim() != 2 || codes->scalar_type() != at::kByte || !block_size(a[2], &block) ||
        !integer(a[3], 0, 255, &fmt) || !integer(a[7], 0, 255, &elem))
        return none();
    const int64_t rows = codes->size(0), cols = 2 * codes->size(1);
    float T = 1.0f;
    const at::Tensor* t_dev = nullptr;
    if (cols % block != 0 || !buffer(a[1], rows * (cols / block), at::kByte)) return none();
    if (!number(a[4], &T) && !(t_dev = buffer(a[4], 4, at::kFloat))) return none();
    const at::Tensor* given = nullptr;
    at::ScalarType type = at::kFloat;
    if (a[6] != Py_None) {
        given = plain(a[6]);
        if (!given || given->numel() < rows * cols) return none();
        type = given->scalar_type();
    } else {
        if (!THPDtype_Check(a[5])) return none();
        type = reinterpret_cast<THPDtype*>(a[5])->scalar_type;
    }
    if (type != at::kFloat && type != at::kBFloat16) return none();
    const at::Tensor out = given ? *given : NewOutputs()({rows, cols}, type, *codes);
    const at::Tensor& scales = THPVariable_Unpack(a[1]);
    int status;
    {
        void* st = stream();
        Unlocked u;
        if (t_dev)
            status = p_dequantize_hier((const uint8_t*)ptr(*codes), (const uint8_t*)ptr(scales), rows, cols, block, elem, fmt,
                                       (const float*)ptr(*t_dev), ptr(out), dtype_code(out), st);
        else
            status = p_dequantize((const uint8_t*)ptr(*codes), (const uint8_t*)ptr(scales), rows, cols, block, elem, fmt, T, ptr(out),
                                  dtype_code(out), st);
    }
    return status != MXQ_OK ? PyLong_FromLong(status) : wrapped(out);
    END_HANDLE_TH_ERRORS
}

// clip_sse(x, scales, block, scale_fmt, tensor_scale, out, elem_fmt)
PyObject* clip_sse(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Input in;
    int fmt, elem;
    float T;
    if (n != 7 || modes_active() || !in.set(a[0], a[2]) || !buffer(a[1], in.blocks, at::kByte) || !integer(a[3], 0, 255, &fmt) ||
        !number(a[4], &T) || !(a[5] == Py_None || buffer(a[5], 4 * in.blocks, at::kFloat)) || !integer(a[6], 0, 255, &elem))
        return none();
    const at::Tensor& scales = THPVariable_Unpack(a[1]);
    const at::Tensor out = a[5] != Py_None ? THPVariable_Unpack(a[5]) : NewOutputs()({in.rows, in.cols / in.block}, at::kFloat, *in.x);
    int status;
    {
        void* st = stream();
        Unlocked u;
        status = p_clip_sse(ptr(*in.x), (const uint8_t*)ptr(scales), in.rows, in.cols, in.block, elem, fmt, T, (float*)ptr(out), in.dt, st);
    }
    return status != MXQ_OK ? PyLong_FromLong(status) : wrapped(out);
    END_HANDLE_TH_ERRORS
}

// histogram(codes, scales, block, elem_fmt), outputs allocated here
PyObject* histogram(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    int block, elem;
    const at::Tensor* codes = (n == 4 && !modes_active()) ? plain(a[0]) : nullptr;
    if (!codes || codes->dim() != 2 || codes->scalar_type() != at::kByte || !block_size(a[2], &block) || !integer(a[3], 0, 255, &elem))
        return none();
    const int64_t rows = codes->size(0), cols = 2 * codes->size(1);
    if (cols % block != 0 || !buffer(a[1], rows * (cols / block), at::kByte)) return none();
    const at::Tensor& scales = THPVariable_Unpack(a[1]);
    NewOutputs new_empty;
    const at::Tensor eh = new_empty({8}, at::kLong, *codes), sh = new_empty({256}, at::kLong, *codes);
    int status;
    {
        void* st = stream();
        Unlocked u;
        status = p_histogram((const uint8_t*)ptr(*codes), (const uint8_t*)ptr(scales), rows, cols, block, elem, (uint64_t*)ptr(eh),
                             (uint64_t*)ptr(sh), st);
    }
    if (status != MXQ_OK) return PyLong_FromLong(status);
    return tuple_of({eh, sh});
    END_HANDLE_TH_ERRORS
}

// new_outputs_direct(): whether outputs made now would be allocated past the dispatcher
PyObject* new_outputs_direct(PyObject*, PyObject*) { return PyBool_FromLong(nothing_watches()); }

// built_for(): what the layouts and signatures compiled in here belong to; mxq.py compares it before use()
PyObject* built_for(PyObject*, PyObject*) { return Py_BuildValue("(ss)", MXQ_CALLS_ABI, MXQ_HEADER_ID); }

// use(address, ...): the library's functions in the order of the declarations above
PyObject* use(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    void* p[8];
    if (n != 8) { PyErr_SetString(PyExc_TypeError, "eight addresses"); return nullptr; }
    for (int i = 0; i < 8; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address"); return nullptr; }
    }
    p_quantize = (decltype(p_quantize))p[0];
    p_quantize_hier = (decltype(p_quantize_hier))p[1];
    p_quantize_batch = (decltype(p_quantize_batch))p[2];
    p_tensor_absmax = (decltype(p_tensor_absmax))p[3];
    p_dequantize = (decltype(p_dequantize))p[4];
    p_dequantize_hier = (decltype(p_dequantize_hier))p[5];
    p_clip_sse = (decltype(p_clip_sse))p[6];
    p_histogram = (decltype(p_histogram))p[7];
    Py_RETURN_NONE;
}

#define MXQ_METHOD(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MXQ_METHOD(quantize), MXQ_METHOD(quantize_hier), MXQ_METHOD(quantize_batch), MXQ_METHOD(tensor_absmax),
                         MXQ_METHOD(dequantize), MXQ_METHOD(clip_sse), MXQ_METHOD(histogram), MXQ_METHOD(use),
                         {"new_outputs_direct", new_outputs_direct, METH_NOARGS, nullptr},
                         {"built_for", built_for, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mxq_calls", "The calls of mxq.py in native code.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__mxq_calls(void) { return PyModule_Create(&module); }
