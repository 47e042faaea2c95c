// Argument marshalling of the short ops in native code, for paper_2604_11947_amd.resbm.
//
// A short op runs for 4-10 us on the device, and the Python checks, pointer and
// stream look-ups and the ctypes call around it took 8.9 us of host time (of 51
// for the four ops of a 256 x 512 stage with their 6 launches at 2.2 us each).
// Each function here takes a library function's address and the op's arguments,
// applies the binding's checks and calls it.  It returns the status, or None for
// anything but plain CUDA tensors that pass every check (subclasses, wrapped
// tensors, wrong types or shapes, no workspace): the caller then goes through
// the Python path, which raises the error or handles the case.  Nothing is kept
// between calls.
#include <torch/csrc/autograd/python_variable.h>

#include <stdint.h>

namespace {

PyObject* g_raw_stream = nullptr;  // torch._C._cuda_getCurrentRawStream

struct Refuse {};  // "not the plain case"
void need(bool ok) {
  if (!ok) throw Refuse();
}

const at::Tensor& tensor(PyObject* o, at::ScalarType t) {
  need(THPVariable_CheckExact(o));
  const at::Tensor& v = THPVariable_Unpack(o);
  need(v.scalar_type() == t && v.is_cuda() && v.layout() == at::kStrided);
  return v;
}
const at::Tensor& matrix(PyObject* o, at::ScalarType t, int64_t rows, int64_t cols) {
  const at::Tensor& v = tensor(o, t);
  need(v.dim() == 2 && v.size(0) == rows && v.size(1) == cols);
  return v;
}
void* packed(PyObject* o, at::ScalarType t, int64_t rows, int64_t cols) {
  const at::Tensor& v = matrix(o, t, rows, cols);
  need(v.is_contiguous());
  return v.data_ptr();
}
void* packed_or_none(PyObject* o, at::ScalarType t, int64_t rows, int64_t cols) {
  return o == Py_None ? nullptr : packed(o, t, rows, cols);
}
// Rows of any stride; ld: the row stride (at least cols for a single row).
void* strided(PyObject* o, at::ScalarType t, int64_t rows, int64_t cols, int64_t* ld) {
  const at::Tensor& v = matrix(o, t, rows, cols);
  need(rows <= 1 || cols <= 0 || v.stride(1) == 1);
  *ld = rows > 1 ? v.stride(0) : std::max(v.stride(0), cols);
  return v.data_ptr();
}
void* strided_or_none(PyObject* o, at::ScalarType t, int64_t rows, int64_t cols, int64_t* ld) {
  *ld = 0;
  return o == Py_None ? nullptr : strided(o, t, rows, cols, ld);
}
struct Bytes {
  void* p;
  size_t n;
};
Bytes workspace(PyObject* o) {
  need(THPVariable_CheckExact(o));
  const at::Tensor& v = THPVariable_Unpack(o);
  need(v.is_cuda());
  return {v.data_ptr(), (size_t)v.numel()};
}
int32_t small_int(PyObject* o) {
  need(PyLong_CheckExact(o));
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(o, &overflow);
  need(!overflow && v >= INT32_MIN && v <= INT32_MAX);
  return (int32_t)v;
}
double real(PyObject* o) {
  need(PyFloat_CheckExact(o));
  return PyFloat_AS_DOUBLE(o);
}
int32_t truth(PyObject* o) {
  need(o == Py_True || o == Py_False);
  return o == Py_True;
}
int32_t dim32(int64_t v) {
  need(v >= 0 && v <= INT32_MAX);
  return (int32_t)v;
}
void* address(PyObject* o) { return PyLong_AsVoidPtr(o); }

// The current stream of t's device, as torch.cuda.current_stream gives it.
void* stream_of(const at::Tensor& t) {
  PyObject* i = PyLong_FromLong(t.get_device());
  PyObject* s = i ? PyObject_CallOneArg(g_raw_stream, i) : nullptr;
  Py_XDECREF(i);
  if (!s) {
    PyErr_Clear();
    throw Refuse();
  }
  void* p = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  return p;
}

template <class F>
PyObject* guarded(F f) {
  try {
    return PyLong_FromLong(f());
  } catch (...) {  // Refuse, or an error of a tensor method: the Python path meets it again
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// Calls fn(args...) without the interpreter lock, as ctypes does.
template <class... P, class... A>
int32_t call(PyObject* fn, int32_t (*)(P...), A... a) {
  auto f = reinterpret_cast<int32_t (*)(P...)>(address(fn));
  int32_t st;
  Py_BEGIN_ALLOW_THREADS
  st = f(a...);
  Py_END_ALLOW_THREADS
  return st;
}

constexpr at::ScalarType F32 = at::kFloat;
at::ScalarType io_type(PyObject* code) { return small_int(code) == 0 ? at::kBFloat16 : at::kFloat; }

typedef int32_t EncFwd(int64_t, int32_t, int32_t, int32_t, const void*, int64_t, const void*, int64_t, const void*,
                       void*, void*, void*, size_t, void*);
typedef int32_t DecFwd(int64_t, int32_t, int32_t, int32_t, const void*, const void*, void*, int64_t, void*, size_t,
                       void*);
typedef int32_t DecBwd(int64_t, int32_t, int32_t, const void*, const void*, const void*, int64_t, const void*, int64_t,
                       void*, void*, int32_t, void*, size_t, void*);
typedef int32_t EncBwd(int64_t, int32_t, int32_t, int32_t, const void*, int64_t, const void*, const void*, const void*,
                       void*, int64_t, void*, int64_t, void*, int32_t, void*, size_t, void*);
typedef int32_t Muon(int32_t, int32_t, void*, const void*, void*, double, double, double, double, int32_t, int32_t,
                     double, double, double, void*, size_t, void*);

// (fn, io_code, x_attn, z, W_e, b, a_save, act, ws)
PyObject* encode_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 9) Py_RETURN_NONE;
  return guarded([&] {
    const at::ScalarType io = io_type(a[1]);
    const at::Tensor &z = tensor(a[3], io), &W = tensor(a[4], F32);
    need(z.dim() == 2 && W.dim() == 2);
    const int64_t T = z.size(0), nn = W.size(0), r = W.size(1);
    int64_t ld_x, ld_z;
    const void* x = strided(a[2], io, T, nn, &ld_x);
    const void* zp = strided(a[3], io, T, nn, &ld_z);
    void* b = packed(a[5], io, T, r);
    const void* w = packed(a[4], F32, nn, r);
    void* s = packed_or_none(a[6], F32, T, r);
    const int32_t act = small_int(a[7]);
    const Bytes ws = workspace(a[8]);
    return call(a[0], (EncFwd*)nullptr, T, dim32(nn), dim32(r), act, x, ld_x, zp, ld_z, w, b, s, ws.p, ws.n,
                stream_of(z));
  });
}

// (fn, io_code, b, W_d, z_tilde, add_identity, ws)
PyObject* decode_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 7) Py_RETURN_NONE;
  return guarded([&] {
    const at::ScalarType io = io_type(a[1]);
    const at::Tensor &b = tensor(a[2], io), &W = tensor(a[3], F32);
    need(b.dim() == 2 && W.dim() == 2);
    const int64_t T = b.size(0), r = W.size(0), nn = W.size(1);
    int64_t ld;
    const void* bp = packed(a[2], io, T, r);
    const void* w = packed(a[3], F32, r, nn);
    void* zt = strided(a[4], io, T, nn, &ld);
    const int32_t add = truth(a[5]);
    const Bytes ws = a[6] == Py_None ? Bytes{nullptr, 0} : workspace(a[6]);
    return call(a[0], (DecFwd*)nullptr, T, dim32(nn), dim32(r), add, bp, w, zt, ld, ws.p, ws.n, stream_of(b));
  });
}

// (fn, io_code, b, W_d, g_zt, g_id, g_b, dW_d, accumulate, ws)
PyObject* decode_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 10) Py_RETURN_NONE;
  return guarded([&] {
    const at::ScalarType io = io_type(a[1]);
    const at::Tensor &b = tensor(a[2], io), &W = tensor(a[3], F32);
    need(b.dim() == 2 && W.dim() == 2);
    const int64_t T = b.size(0), r = W.size(0), nn = W.size(1);
    int64_t ld_g, ld_i;
    const void* bp = packed(a[2], io, T, r);
    const void* w = packed(a[3], F32, r, nn);
    const void* g = strided(a[4], io, T, nn, &ld_g);
    const void* gi = strided_or_none(a[5], io, T, nn, &ld_i);
    void* gb = packed(a[6], io, T, r);
    void* dW = packed(a[7], F32, r, nn);
    const int32_t acc = truth(a[8]);
    const Bytes ws = workspace(a[9]);
    return call(a[0], (DecBwd*)nullptr, T, dim32(nn), dim32(r), bp, w, g, ld_g, gi, ld_i, gb, dW, acc, ws.p, ws.n,
                stream_of(THPVariable_Unpack(a[4])));
  });
}

// (fn, io_code, z, W_e, a_save, g_b, g_z, dW_e, g_x, act, accumulate, ws)
PyObject* encode_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 12) Py_RETURN_NONE;
  return guarded([&] {
    const at::ScalarType io = io_type(a[1]);
    const at::Tensor &z = tensor(a[2], io), &W = tensor(a[3], F32);
    need(z.dim() == 2 && W.dim() == 2);
    const int64_t T = z.size(0), nn = W.size(0), r = W.size(1);
    int64_t ld_z, ld_gz, ld_gx;
    const void* zp = strided(a[2], io, T, nn, &ld_z);
    const void* w = packed(a[3], F32, nn, r);
    const void* s = packed_or_none(a[4], F32, T, r);
    const void* gb = packed(a[5], io, T, r);
    void* gz = strided(a[6], io, T, nn, &ld_gz);
    void* dW = packed(a[7], F32, nn, r);
    void* gx = strided_or_none(a[8], io, T, nn, &ld_gx);
    const int32_t act = small_int(a[9]), acc = truth(a[10]);
    const Bytes ws = workspace(a[11]);
    return call(a[0], (EncBwd*)nullptr, T, dim32(nn), dim32(r), act, zp, ld_z, w, s, gb, gz, ld_gz, gx, ld_gx, dW, acc,
                ws.p, ws.n, stream_of(z));
  });
}

// (fn, W, G, M, lr, momentum, weight_decay, scale, nesterov, steps, (a, b, c), ws)
PyObject* muon_update(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 12) Py_RETURN_NONE;
  return guarded([&] {
    const at::Tensor& W = tensor(a[1], F32);
    need(W.dim() == 2);
    const int64_t p = W.size(0), q = W.size(1);
    void* w = packed(a[1], F32, p, q);
    const void* g = packed(a[2], F32, p, q);
    void* m = packed_or_none(a[3], F32, p, q);
    const int32_t nest = truth(a[8]), steps = small_int(a[9]);
    need(PyTuple_CheckExact(a[10]) && PyTuple_GET_SIZE(a[10]) == 3);
    double c[3];
    for (int i = 0; i < 3; ++i) c[i] = real(PyTuple_GET_ITEM(a[10], i));
    const Bytes ws = workspace(a[11]);
    return call(a[0], (Muon*)nullptr, dim32(p), dim32(q), w, g, m, real(a[4]), real(a[5]), real(a[6]), real(a[7]), nest,
                steps, c[0], c[1], c[2], ws.p, ws.n, stream_of(W));
  });
}

PyObject* init(PyObject*, PyObject* raw_stream) {
  Py_INCREF(raw_stream);
  Py_XDECREF(g_raw_stream);
  g_raw_stream = raw_stream;
  Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(encode_fwd), FAST(decode_fwd), FAST(decode_bwd), FAST(encode_bwd), FAST(muon_update),
                         {"init", init, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
