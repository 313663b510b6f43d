// The single-layer calls of binding.py from Python, without ctypes: a call of a few microseconds on the GPU is bound by its
// host time, and of that the launch itself takes 3.0 us; attribute reads, argument conversion and the foreign-function
// interface took another 1.6 (ReLU) to 3 (convolution), here some 0.4.
//
// Every function takes the arguments of the binding's function of that name, positionally, with the stream last, and
// returns the library's status. It returns None, having done nothing, for whatever is not the plain case (a stream given,
// tensors of a subclass, integers or paddings or quantization records of other types): the binding then makes the same call
// through ctypes, which accepts or refuses it.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <dlfcn.h>
#include <stddef.h>

#include "../../include/small.h"

namespace {

PyTypeObject *quant_type = nullptr;        // binding.small_quant

#define SMALL_FUNCTIONS(X)                                                                                                        \
    X(small_pack) X(small_unpack) X(small_conv2d) X(small_dwconv2d) X(small_pool2d) X(small_relu) X(small_add) X(small_dense)     \
    X(small_pack_u8) X(small_unpack_u8) X(small_conv2d_u8) X(small_dwconv2d_u8) X(small_dense_u8) X(small_pool2d_u8) X(small_relu_u8)
struct Library {
#define X(f) decltype(&::f) f = nullptr;
    SMALL_FUNCTIONS(X)
#undef X
} lib;

// Reads one call's arguments; `plain` turns false at the first that is not the plain case.
struct Reader {
    PyObject *const *a;
    bool plain, error = false;
    Py_buffer quant = {};

    Reader(PyObject *const *args, Py_ssize_t n, Py_ssize_t expected) : a(args), plain(n == expected && lib.small_relu && args[n - 1] == Py_None) {}
    ~Reader()
    {
        if (quant.obj) PyBuffer_Release(&quant);
    }
    unsigned long number(int k)
    {
        if (!plain) return 0;
        if (!PyLong_CheckExact(a[k])) {
            plain = false;
            return 0;
        }
        return PyLong_AsUnsignedLongMask(a[k]);          // (as ctypes converts: modulo the type's range)
    }
    int i(int k) { return (int)number(k); }
    small_pad pad(int k)
    {
        int side[4] = {0, 0, 0, 0};
        if (!plain) return {0, 0, 0, 0};
        PyObject *p = a[k];
        if (!PyTuple_CheckExact(p) || PyTuple_GET_SIZE(p) > 4) {
            plain = false;
            return {0, 0, 0, 0};
        }
        for (Py_ssize_t j = 0; j < PyTuple_GET_SIZE(p); ++j) {
            PyObject *v = PyTuple_GET_ITEM(p, j);
            if (!PyLong_CheckExact(v)) plain = false;
            else side[j] = (int)PyLong_AsUnsignedLongMask(v);
        }
        return {side[0], side[1], side[2], side[3]};
    }
    const small_quant *q(int k)
    {
        if (!plain) return nullptr;
        if (Py_TYPE(a[k]) != quant_type || PyObject_GetBuffer(a[k], &quant, PyBUF_SIMPLE) != 0 || quant.len != (Py_ssize_t)sizeof(small_quant)) {
            PyErr_Clear();
            plain = false;
            return nullptr;
        }
        return static_cast<const small_quant *>(quant.buf);
    }
    template <typename T>
    T *tensor(int k, at::ScalarType type, const char *refusal)
    {
        if (!plain || error || a[k] == Py_None) return nullptr;
        if (!THPVariable_CheckExact(a[k])) {
            plain = false;
            return nullptr;
        }
        const at::Tensor &t = THPVariable_Unpack(a[k]);
        if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) {
            PyErr_SetString(PyExc_TypeError, refusal);
            error = true;
            return nullptr;
        }
        return static_cast<T *>(t.data_ptr());
    }
    float *f32(int k) { return tensor<float>(k, at::kFloat, "expected a contiguous float32 CUDA tensor"); }
    unsigned char *u8(int k) { return tensor<unsigned char>(k, at::kByte, "expected a contiguous uint8 CUDA tensor"); }
    int *i32(int k) { return tensor<int>(k, at::kInt, "expected a contiguous int32 CUDA tensor"); }

    // The call, if everything was plain, on the current stream of the current device; without the interpreter lock, which ctypes
    // does not hold either.
    template <typename F>
    PyObject *call(F f)
    {
        if (error) return nullptr;
        if (!plain) Py_RETURN_NONE;
        void *stream = c10::hip::getCurrentHIPStream().stream();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = f(stream);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    }
};

// The other arguments are read before the tensors, so that a call that is not plain raises nothing here.
#define ENTRY(name, n_args, ...)                                              \
    PyObject *name(PyObject *, PyObject *const *args, Py_ssize_t n)           \
    {                                                                         \
        HANDLE_TH_ERRORS                                                      \
        Reader r(args, n, n_args);                                            \
        __VA_ARGS__                                                           \
        END_HANDLE_TH_ERRORS                                                  \
    }

#define LAYOUT(name, fn, tensor)                                                                                    \
    ENTRY(name, 8, const int N = r.i(2), C = r.i(3), H = r.i(4), W = r.i(5), Cb = r.i(6);                           \
          auto *src = r.tensor(0); auto *dst = r.tensor(1);                                                         \
          return r.call([&](void *s) { return lib.fn(src, dst, N, C, H, W, Cb, s); });)
LAYOUT(pack, small_pack, f32)
LAYOUT(unpack, small_unpack, f32)
LAYOUT(pack_u8, small_pack_u8, u8)
LAYOUT(unpack_u8, small_unpack_u8, u8)

ENTRY(conv2d, 15, const int N = r.i(3), Ci = r.i(4), Co = r.i(5), H = r.i(6), W = r.i(7), kh = r.i(8), kw = r.i(9), st = r.i(10);
      const small_pad pad = r.pad(11); const int Cib = r.i(12), Cob = r.i(13);
      auto *x = r.f32(0); auto *w = r.f32(1); auto *y = r.f32(2);
      return r.call([&](void *s) { return lib.small_conv2d(x, w, y, N, Ci, Co, H, W, kh, kw, st, pad, Cib, Cob, s); });)
ENTRY(conv2d_u8, 17, const int N = r.i(3), Ci = r.i(4), Co = r.i(5), H = r.i(6), W = r.i(7), kh = r.i(8), kw = r.i(9), st = r.i(10);
      const small_pad pad = r.pad(11); const int Cib = r.i(12), Cob = r.i(13); const small_quant *q = r.q(14);
      auto *x = r.u8(0); auto *w = r.u8(1); auto *y = r.u8(2); auto *sums = r.i32(15);
      return r.call([&](void *s) { return lib.small_conv2d_u8(x, w, y, N, Ci, Co, H, W, kh, kw, st, pad, Cib, Cob, q, sums, s); });)
ENTRY(dwconv2d, 13, const int N = r.i(3), C = r.i(4), H = r.i(5), W = r.i(6), kh = r.i(7), kw = r.i(8), st = r.i(9);
      const small_pad pad = r.pad(10); const int Cb = r.i(11);
      auto *x = r.f32(0); auto *w = r.f32(1); auto *y = r.f32(2);
      return r.call([&](void *s) { return lib.small_dwconv2d(x, w, y, N, C, H, W, kh, kw, st, pad, Cb, s); });)
ENTRY(dwconv2d_u8, 14, const int N = r.i(3), C = r.i(4), H = r.i(5), W = r.i(6), kh = r.i(7), kw = r.i(8), st = r.i(9);
      const small_pad pad = r.pad(10); const int Cb = r.i(11); const small_quant *q = r.q(12);
      auto *x = r.u8(0); auto *w = r.u8(1); auto *y = r.u8(2);
      return r.call([&](void *s) { return lib.small_dwconv2d_u8(x, w, y, N, C, H, W, kh, kw, st, pad, Cb, q, s); });)

#define POOL(name, fn, tensor)                                                                                                  \
    ENTRY(name, 13, const int N = r.i(2), C = r.i(3), H = r.i(4), W = r.i(5), kh = r.i(6), kw = r.i(7), st = r.i(8);            \
          const small_pad pad = r.pad(9); const int Cb = r.i(10), mode = r.i(11);                                               \
          auto *x = r.tensor(0); auto *y = r.tensor(1);                                                                         \
          return r.call([&](void *s) { return lib.fn(x, y, N, C, H, W, kh, kw, st, pad, Cb, mode, s); });)
POOL(pool2d, small_pool2d, f32)
POOL(pool2d_u8, small_pool2d_u8, u8)

ENTRY(relu, 4, const size_t n_el = r.number(2); auto *x = r.f32(0); auto *y = r.f32(1);
      return r.call([&](void *s) { return lib.small_relu(x, y, n_el, s); });)
ENTRY(relu_u8, 5, const size_t n_el = r.number(2); const int z = r.i(3); auto *x = r.u8(0); auto *y = r.u8(1);
      return r.call([&](void *s) { return lib.small_relu_u8(x, y, n_el, z, s); });)
ENTRY(add, 5, const size_t n_el = r.number(3); auto *x = r.f32(0); auto *b = r.f32(1); auto *y = r.f32(2);
      return r.call([&](void *s) { return lib.small_add(x, b, y, n_el, s); });)
ENTRY(dense, 9, const int N = r.i(3), Ci = r.i(4), Co = r.i(5), Cib = r.i(6), Cob = r.i(7);
      auto *x = r.f32(0); auto *w = r.f32(1); auto *y = r.f32(2);
      return r.call([&](void *s) { return lib.small_dense(x, w, y, N, Ci, Co, Cib, Cob, s); });)
ENTRY(dense_u8, 11, const int N = r.i(3), Ci = r.i(4), Co = r.i(5), Cib = r.i(6), Cob = r.i(7); const small_quant *q = r.q(8);
      auto *x = r.u8(0); auto *w = r.u8(1); auto *y = r.u8(2); auto *sums = r.i32(9);
      return r.call([&](void *s) { return lib.small_dense_u8(x, w, y, N, Ci, Co, Cib, Cob, q, sums, s); });)

// bind(handle of the loaded library, the binding's small_quant)
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 2 || !PyLong_Check(args[0]) || !PyType_Check(args[1])) {
        PyErr_SetString(PyExc_TypeError, "bind(handle, small_quant)");
        return nullptr;
    }
    void *handle = PyLong_AsVoidPtr(args[0]);
    if (!handle) return nullptr;
#define X(f)                                                        \
    lib.f = reinterpret_cast<decltype(&::f)>(dlsym(handle, #f));    \
    if (!lib.f) {                                                   \
        lib.small_relu = nullptr;                                   \
        PyErr_SetString(PyExc_AttributeError, #f);                  \
        return nullptr;                                             \
    }
    SMALL_FUNCTIONS(X)
#undef X
    Py_INCREF(args[1]);                    // (kept for the module's life)
    quant_type = reinterpret_cast<PyTypeObject *>(args[1]);
    Py_RETURN_NONE;
}

#define METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(bind), METHOD(pack), METHOD(unpack), METHOD(pack_u8), METHOD(unpack_u8), METHOD(conv2d), METHOD(conv2d_u8),
                         METHOD(dwconv2d), METHOD(dwconv2d_u8), METHOD(pool2d), METHOD(pool2d_u8), METHOD(relu), METHOD(relu_u8), METHOD(add),
                         METHOD(dense), METHOD(dense_u8), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() { return PyModule_Create(&module); }
