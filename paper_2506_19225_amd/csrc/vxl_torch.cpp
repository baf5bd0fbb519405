// The hot entry points of include/vxl.h as Python functions over torch tensors: argument marshalling only.
// A small call is bound by the host: through ctypes, seven tensors asked for is_cuda, is_contiguous and data_ptr and
// thirteen arguments converted took 2.5 of the 9.0 us that a generated token's call took to submit, which is 6.5 so (two
// launches); the four calls of a prompt of 576 tokens 25.7 -> 17.1, a question's three on 16k tokens 22.5 -> 16.2.
//
// Arguments in the order of the C functions, without the sizes, which are read off the tensors; last the stream, which
// vxl._stream makes a handle of when all others are found good.  What an argument may be goes by its position alone (the
// kinds at each function below): an object of another kind is refused, never taken for an address.  The result is the
// vxl_status.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "vxl.h"

namespace {

// The functions of the library that vxl.lib() loaded, as setup() is given them: linked against it, the binding of a second
// copy in the process called the first copy's library, and one of another path than its own was never called.
#define VXL_PATH(X)                                                                                               \
    X(chunk_prefill) X(chunk_score_topk) X(chunk_score_topk_mass) X(gather_bilevel_kv) X(pool_sparse_kv)          \
    X(gather_bilevel_kv_pooled) X(bilevel_decode) X(bilevel_decode_inplace)

// Of one module object: a vxl.py that is loaded twice has two.
struct State {
    PyObject *desc_type, *handle_type, *stream_of;
#define VXL_DECLARE(name) decltype(&vxl_##name) name;
    VXL_PATH(VXL_DECLARE)
};

// Kinds of an argument: a layout's c_void_p (or a number or None, the library's to refuse); the descriptor; a tensor (its
// data pointer; a contiguous CUDA tensor or AssertionError) or None, a null pointer; a number.  Python does not pass
// kNumel, the number of elements of the tensor before it (0 for None), and size(i, d), dimension d of its argument i.
enum Kind { kLayout, kDesc, kTensor, kInt, kNumel, kSize };
constexpr int size(int arg, int dim) { return kSize | arg << 8 | dim << 16; }

// A number that an object answers with (a new reference, or null where it raised).
bool take(PyObject* r, long long* out) {
    if (!r) return false;
    *out = (long long)PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

// Pointer of an object that is not a torch.Tensor but answers like one.
bool like_tensor(PyObject* o, long long* out) {
    PyObject* cuda = PyObject_GetAttrString(o, "is_cuda");
    if (!cuda) return false;
    int ok = PyObject_IsTrue(cuda);
    Py_DECREF(cuda);
    PyObject* r = ok > 0 ? PyObject_CallMethod(o, "is_contiguous", nullptr) : nullptr;
    if (ok < 0 || (ok > 0 && !r)) return false;
    if (r) {
        ok = PyObject_IsTrue(r);
        Py_DECREF(r);
        if (ok < 0) return false;
    }
    if (!ok) {
        PyErr_SetString(PyExc_AssertionError, "device tensors must be contiguous CUDA tensors");
        return false;
    }
    return take(PyObject_CallMethod(o, "data_ptr", nullptr), out);
}

bool size_of(PyObject* o, int d, long long* out) {
    if (THPVariable_Check(o)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (d >= t.dim()) { PyErr_SetString(PyExc_IndexError, "tuple index out of range"); return false; }
        *out = t.size(d);
        return true;
    }
    PyObject* shape = PyObject_GetAttrString(o, "shape");
    if (!shape) return false;
    PyObject* r = PySequence_GetItem(shape, d);
    Py_DECREF(shape);
    return take(r, out);
}

bool numel_of(PyObject* o, long long* out) {
    if (o == Py_None) { *out = 0; return true; }
    if (THPVariable_Check(o)) { *out = THPVariable_Unpack(o).numel(); return true; }
    return take(PyObject_CallMethod(o, "numel", nullptr), out);
}

// The memory of a ctypes object.
bool memory_of(PyObject* o, void** out) {
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) < 0) return false;
    *out = view.buf;
    PyBuffer_Release(&view);                                  // (the object, which the caller holds, owns it)
    return true;
}

bool refuse(PyObject* o, const char* what) {
    PyErr_Format(PyExc_TypeError, "%s expected, not '%.100s'", what, Py_TYPE(o)->tp_name);
    return false;
}

bool int_of(PyObject* o, long long* out) {
    if (!PyLong_Check(o)) return refuse(o, "a number");
    *out = (long long)PyLong_AsUnsignedLongLongMask(o);
    return !PyErr_Occurred();
}

bool tensor_of(PyObject* o, long long* out) {
    if (o == Py_None) { *out = 0; return true; }
    if (!THPVariable_Check(o)) return like_tensor(o, out);
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) {
        PyErr_SetString(PyExc_AssertionError, "device tensors must be contiguous CUDA tensors");
        return false;
    }
    *out = (long long)t.data_ptr();
    return true;
}

bool desc_of(const State& st, PyObject* o, long long* out) {
    void* p = nullptr;
    if (!PyObject_TypeCheck(o, (PyTypeObject*)st.desc_type)) return refuse(o, "a descriptor");
    if (!memory_of(o, &p)) return false;
    *out = (long long)p;
    return true;
}

bool layout_of(const State& st, PyObject* o, long long* out) {
    void* p = nullptr;
    if (o == Py_None) { *out = 0; return true; }
    if (PyLong_Check(o)) return int_of(o, out);
    if (!PyObject_TypeCheck(o, (PyTypeObject*)st.handle_type)) return refuse(o, "a layout's handle");
    if (!memory_of(o, &p)) return false;
    *out = (long long)*(void**)p;
    return true;
}

constexpr bool passed(int kind) { return kind < kNumel; }

// The argument of this kind: the next of Python's, or a number read off one.
template <int KIND>
bool convert(const State& st, PyObject* const* args, int* next, long long* out) {
    if constexpr ((KIND & 255) == kSize) return size_of(args[KIND >> 8 & 255], KIND >> 16, out);
    else if constexpr (KIND == kNumel) return numel_of(args[*next - 1], out);
    else if constexpr (KIND == kLayout) return layout_of(st, args[(*next)++], out);
    else if constexpr (KIND == kDesc) return desc_of(st, args[(*next)++], out);
    else if constexpr (KIND == kTensor) return tensor_of(args[(*next)++], out);
    else return int_of(args[(*next)++], out);
}

// f over the library's functions, the arguments of these kinds and the stream.
template <int... KINDS, typename F>
PyObject* call(PyObject* self, PyObject* const* args, Py_ssize_t n, F f) {
    const State& st = *(const State*)PyModule_GetState(self);
    constexpr int given = (passed(KINDS) + ...) + 1;
    if (n != given) { PyErr_Format(PyExc_TypeError, "%d arguments expected, %zd given", given, n); return nullptr; }
    if (!st.desc_type) { PyErr_SetString(PyExc_RuntimeError, "setup() has not been called"); return nullptr; }
    long long a[sizeof...(KINDS) + 1], *out = a;
    int next = 0;
    try {
        if (!(convert<KINDS>(st, args, &next, out++) && ...)) return nullptr;
    } catch (const std::exception& e) {                       // (a tensor without memory)
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    PyObject* s = PyObject_CallFunctionObjArgs(st.stream_of, args[n - 1], nullptr);
    if (!s) return nullptr;
    *out = s == Py_None ? 0 : (long long)PyLong_AsUnsignedLongLongMask(s);
    Py_DECREF(s);
    if (PyErr_Occurred()) return nullptr;
    vxl_status status;
    Py_BEGIN_ALLOW_THREADS
    status = f(st, a);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

template <typename T> T* ptr(long long a) { return (T*)a; }
const vxl_layout* lay(long long a) { return (const vxl_layout*)a; }
const vxl_attn_desc* desc(long long a) { return (const vxl_attn_desc*)a; }

PyObject* chunk_prefill(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    return call<kLayout, kDesc, kTensor, kTensor, kTensor, kTensor, kTensor, kTensor, kNumel>(
        self, args, n, [](const State& lib, const long long* a) {
        return lib.chunk_prefill(lay(a[0]), desc(a[1]), ptr<void>(a[2]), ptr<void>(a[3]), ptr<void>(a[4]), ptr<void>(a[5]),
                                 ptr<float>(a[6]), ptr<void>(a[7]), (size_t)a[8], (vxl_stream)a[9]);
    });
}
PyObject* chunk_score_topk(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    return call<kLayout, kDesc, kTensor, size(2, 0), size(2, 1), kTensor, kInt, kTensor, kInt, kTensor, kTensor, kTensor, kTensor,
                kNumel>(
        self, args, n, [](const State& lib, const long long* a) {
        return lib.chunk_score_topk(lay(a[0]), desc(a[1]), ptr<void>(a[2]), (int32_t)a[3], (int32_t)a[4], ptr<void>(a[5]),
                                    (int32_t)a[6], ptr<float>(a[7]), (int32_t)a[8], ptr<int32_t>(a[9]), ptr<uint8_t>(a[10]),
                                    ptr<float>(a[11]), ptr<void>(a[12]), (size_t)a[13], (vxl_stream)a[14]);
    });
}
PyObject* chunk_score_topk_mass(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    return call<kLayout, kDesc, kTensor, size(2, 0), size(2, 1), kTensor, kInt, kTensor, kTensor, kTensor, kTensor, kNumel>(
        self, args, n, [](const State& lib, const long long* a) {
        return lib.chunk_score_topk_mass(lay(a[0]), desc(a[1]), ptr<void>(a[2]), (int32_t)a[3], (int32_t)a[4], ptr<void>(a[5]),
                                         (int32_t)a[6], ptr<int32_t>(a[7]), ptr<uint8_t>(a[8]), ptr<float>(a[9]),
                                         ptr<void>(a[10]), (size_t)a[11], (vxl_stream)a[12]);
    });
}
PyObject* gather_bilevel_kv(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    return call<kLayout, kDesc, kTensor, kTensor, kTensor, size(5, 0), kTensor, kTensor, size(5, 2), kTensor, kTensor>(
        self, args, n, [](const State& lib, const long long* a) {
        return lib.gather_bilevel_kv(lay(a[0]), desc(a[1]), ptr<void>(a[2]), ptr<void>(a[3]), ptr<uint8_t>(a[4]), (int32_t)a[5],
                                     ptr<void>(a[6]), ptr<void>(a[7]), (int32_t)a[8], ptr<int32_t>(a[9]), ptr<int32_t>(a[10]),
                                     (vxl_stream)a[11]);
    });
}
PyObject* pool_sparse_kv(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    return call<kLayout, kDesc, kTensor, kTensor, kTensor, kTensor>(
        self, args, n, [](const State& lib, const long long* a) {
        return lib.pool_sparse_kv(lay(a[0]), desc(a[1]), ptr<void>(a[2]), ptr<void>(a[3]), ptr<void>(a[4]), ptr<void>(a[5]),
                                  (vxl_stream)a[6]);
    });
}
PyObject* gather_bilevel_kv_pooled(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    return call<kLayout, kDesc, kTensor, kTensor, kTensor, kTensor, kTensor, size(7, 0), kTensor, kTensor, size(7, 2), kTensor, kTensor>(
        self, args, n, [](const State& lib, const long long* a) {
        return lib.gather_bilevel_kv_pooled(lay(a[0]), desc(a[1]), ptr<void>(a[2]), ptr<void>(a[3]), ptr<void>(a[4]),
                                            ptr<void>(a[5]), ptr<uint8_t>(a[6]), (int32_t)a[7], ptr<void>(a[8]), ptr<void>(a[9]),
                                            (int32_t)a[10], ptr<int32_t>(a[11]), ptr<int32_t>(a[12]), (vxl_stream)a[13]);
    });
}
PyObject* bilevel_decode(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    return call<kDesc, kTensor, size(1, 0), size(1, 1), kTensor, kTensor, size(2, 2), kTensor, kTensor, kTensor, kTensor, kNumel>(
        self, args, n, [](const State& lib, const long long* a) {
        return lib.bilevel_decode(desc(a[0]), ptr<void>(a[1]), (int32_t)a[2], (int32_t)a[3], ptr<void>(a[4]), ptr<void>(a[5]),
                                  (int32_t)a[6], ptr<int32_t>(a[7]), ptr<void>(a[8]), ptr<float>(a[9]), ptr<void>(a[10]),
                                  (size_t)a[11], (vxl_stream)a[12]);
    });
}
PyObject* bilevel_decode_inplace(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    return call<kLayout, kDesc, kTensor, size(2, 0), size(2, 1), kTensor, kTensor, kTensor, kTensor, kTensor, kInt, kInt, kTensor,
                kTensor, kTensor, kTensor, kNumel>(
        self, args, n, [](const State& lib, const long long* a) {
        return lib.bilevel_decode_inplace(lay(a[0]), desc(a[1]), ptr<void>(a[2]), (int32_t)a[3], (int32_t)a[4], ptr<void>(a[5]),
                                          ptr<void>(a[6]), ptr<void>(a[7]), ptr<void>(a[8]), ptr<uint8_t>(a[9]), (int32_t)a[10],
                                          (int32_t)a[11], ptr<void>(a[12]), ptr<float>(a[13]), ptr<int32_t>(a[14]),
                                          ptr<void>(a[15]), (size_t)a[16], (vxl_stream)a[17]);
    });
}
// setup(type of the descriptor, type of a layout's handle, vxl._stream, the addresses of VXL_PATH)
PyObject* setup(PyObject* self, PyObject* const* args, Py_ssize_t n) {
#define VXL_COUNT(name) + 1
    if (n != 3 VXL_PATH(VXL_COUNT) || !PyType_Check(args[0]) || !PyType_Check(args[1]) || !PyCallable_Check(args[2])) {
        PyErr_SetString(PyExc_TypeError, "two types, a function and the library's addresses expected");
        return nullptr;
    }
    for (int i = 3; i < n; ++i)
        if (!PyLong_Check(args[i]) || !PyLong_AsVoidPtr(args[i])) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "an address expected");
            return nullptr;
        }
    State& st = *(State*)PyModule_GetState(self);
    int i = 3;
#define VXL_TAKE(name) st.name = (decltype(st.name))PyLong_AsVoidPtr(args[i++]);
    VXL_PATH(VXL_TAKE)
    PyObject** to[] = {&st.desc_type, &st.handle_type, &st.stream_of};
    for (int j = 0; j < 3; ++j) {
        Py_INCREF(args[j]);
        Py_XSETREF(*to[j], args[j]);
    }
    Py_RETURN_NONE;
}

int traverse(PyObject* self, visitproc visit, void* arg) {
    const State* st = (const State*)PyModule_GetState(self);
    if (!st) return 0;
    Py_VISIT(st->desc_type);
    Py_VISIT(st->handle_type);
    Py_VISIT(st->stream_of);
    return 0;
}
int clear(PyObject* self) {
    State* st = (State*)PyModule_GetState(self);
    if (!st) return 0;
    Py_CLEAR(st->desc_type);
    Py_CLEAR(st->handle_type);
    Py_CLEAR(st->stream_of);
    return 0;
}

int exec(PyObject* self) { return PyModule_AddStringConstant(self, "torch_version", VXL_TORCH_VERSION); }

#define VXL_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr},
PyMethodDef methods[] = {VXL_METHOD(setup) VXL_PATH(VXL_METHOD){nullptr, nullptr, 0, nullptr}};
PyModuleDef_Slot slots[] = {{Py_mod_exec, (void*)exec}, {0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_vxl_torch", nullptr, sizeof(State), methods, slots, traverse, clear, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__vxl_torch(void) { return PyModuleDef_Init(&module); }
