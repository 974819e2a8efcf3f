// The Python face of the C ABI: one native function per tensor-taking entry point, called by binding.py.
//
// A layer call of a few microseconds of GPU time is bound by what the host does per launch.  Marshalled with ctypes
// (five tensors, each asked for device, contiguity, type, size and address through Python attributes, then a foreign
// call) a call cost 8 to 9 us of host time, twice the launch itself; read straight from the tensor objects it is
// a few tenths of a microsecond.
//
// For a tensor, the facts the C side cannot see are checked here, because a mismatch would become an out-of-bounds
// access on the device: it must live on a GPU, be contiguous, have the element type the call reads and hold at least
// as many elements as the descriptor asks for (ValueError); a structure must be of its own ctypes class (TypeError).  An
// integer is taken as a raw device address, None as NULL.  The functions return the glowmi_status; binding.py turns it into an exception.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>

#include "../../include/glowmi.h"

namespace {

struct Refused {};                       // a Python exception is set

[[noreturn]] void refuse(PyObject* type, const std::string& message) {
  PyErr_SetString(type, message.c_str());
  throw Refused{};
}

// ---- arguments ------------------------------------------------------------------------------------------
long long integer(PyObject* o) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw Refused{};
  return v;
}

int32_t int32_of(PyObject* o) { return (int32_t)integer(o); }

// An extent that tensors are measured against: cut to 32 bits it would let a tensor pass that is too small.
int32_t extent(PyObject* o, const char* what) {
  const long long v = integer(o);
  if (v != (int32_t)v) refuse(PyExc_ValueError, std::string(what) + ": " + std::to_string(v) + " is not a 32-bit integer");
  return (int32_t)v;
}

float number(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Refused{};
  return (float)v;
}

const at::Tensor& tensor_of(PyObject* o, const char* what) {
  if (!THPVariable_Check(o)) refuse(PyExc_TypeError, std::string(what) + ": expected a tensor, an address or None");
  return THPVariable_Unpack(o);
}

const char* type_name(at::ScalarType t) {
  return t == at::kFloat ? "float32" : t == at::kChar ? "int8" : t == at::kInt ? "int32" : c10::toString(t);
}

// Device address of a tensor of `type` with at least `count` elements; NULL for None; a raw address as it is.
void* address(PyObject* o, at::ScalarType type, long long count, const char* what) {
  if (o == Py_None) return nullptr;
  if (PyLong_Check(o)) {
    void* p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw Refused{};
    return p;
  }
  const at::Tensor& t = tensor_of(o, what);
  if (!t.is_cuda())
    refuse(PyExc_ValueError, std::string(what) + ": expected a device tensor, got one on " + t.device().str());
  if (!t.is_contiguous()) refuse(PyExc_ValueError, std::string(what) + ": tensor is not contiguous");
  if (t.scalar_type() != type)
    refuse(PyExc_ValueError, std::string(what) + ": expected " + type_name(type) + ", got " + type_name(t.scalar_type()));
  if (t.numel() < count)
    refuse(PyExc_ValueError, std::string(what) + ": " + std::to_string(t.numel()) + " elements, the call needs " +
                                 std::to_string(count));
  return t.data_ptr();
}

// A buffer of bytes (workspace, arena, planes): any element type.
struct Bytes {
  void* p = nullptr;
  size_t n = 0;
};
Bytes bytes_of(PyObject* o, const char* what, size_t need = 0) {
  Bytes b;
  if (o == Py_None) return b;
  const at::Tensor& t = tensor_of(o, what);
  if (!t.is_cuda() || !t.is_contiguous())
    refuse(PyExc_ValueError, std::string(what) + ": expected a contiguous device tensor");
  b.n = (size_t)t.numel() * t.element_size();
  if (need && b.n < need)
    refuse(PyExc_ValueError, std::string(what) + ": " + std::to_string(b.n) + " bytes, the filter's planes take " +
                                 std::to_string(need));
  b.p = t.data_ptr();
  return b;
}

// hipStream_t: a raw handle, an object with a cuda_stream handle, or torch's current stream for None.
hipStream_t stream_of(PyObject* o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  if (PyLong_Check(o)) return static_cast<hipStream_t>(PyLong_AsVoidPtr(o));
  PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
  if (!h) throw Refused{};
  void* p = PyLong_AsVoidPtr(h);
  Py_DECREF(h);
  if (!p && PyErr_Occurred()) throw Refused{};
  return static_cast<hipStream_t>(p);
}

// binding.py's ctypes classes, handed over when it loads this module (structure_types below).
PyObject *g_conv_desc = nullptr, *g_qparam = nullptr, *g_seq_layer = nullptr;

void check_type(PyObject* o, PyObject* type, const char* name) {
  if (!type) refuse(PyExc_RuntimeError, "structure types not set");
  if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(type)))
    refuse(PyExc_TypeError, std::string("expected a ") + name + ", got " + Py_TYPE(o)->tp_name);
}

// The memory of a ctypes structure (or array of them), as the C type it mirrors.
template <typename T>
struct View {
  Py_buffer buf;
  size_t count;
  explicit View(PyObject* o) {
    if (PyObject_GetBuffer(o, &buf, PyBUF_SIMPLE) != 0) throw Refused{};
    count = (size_t)buf.len / sizeof(T);
    if (buf.len == 0 || buf.len % sizeof(T) != 0) {
      PyBuffer_Release(&buf);
      refuse(PyExc_TypeError, "argument is not the structure this call takes");
    }
  }
  ~View() { PyBuffer_Release(&buf); }
  View(const View&) = delete;
  const T* get() const { return static_cast<const T*>(buf.buf); }
};

PyObject* checked_desc(PyObject* o) {
  check_type(o, g_conv_desc, "ConvDesc");
  return o;
}

PyObject* checked_layers(PyObject* o) {              // a ctypes array of SeqLayer
  PyObject* item = PyObject_GetAttrString(o, "_type_");
  if (!item) PyErr_Clear();
  const int ok = item && g_seq_layer && PyType_Check(item) ? PyObject_IsSubclass(item, g_seq_layer) : 0;
  Py_XDECREF(item);
  if (ok < 0) throw Refused{};
  if (!ok) refuse(PyExc_TypeError, std::string("expected an array of SeqLayer (seq_layers), got ") + Py_TYPE(o)->tp_name);
  return o;
}

glowmi_qparam qparam_of(PyObject* o) {
  check_type(o, g_qparam, "QParam");
  View<glowmi_qparam> v(o);
  return *v.get();
}

// Element counts of a descriptor's input, filter and output; zeros when the library will reject it.
struct Counts {
  long long x = 0, w = 0, y = 0;
  explicit Counts(const glowmi_conv_desc& d) {
    int32_t oh = 0, ow = 0;
    if (glowmi_conv_out_shape(&d, &oh, &ow) != GLOWMI_OK) return;
    x = (long long)d.n * d.h * d.w * d.c;
    w = (long long)d.k * d.r * d.s * (d.c / d.groups);
    y = (long long)d.n * oh * ow * d.k;
  }
};

constexpr at::ScalarType F32 = at::kFloat, I8 = at::kChar, I32 = at::kInt;

const float* in_f32(PyObject* o, long long n, const char* what) { return static_cast<const float*>(address(o, F32, n, what)); }
float* out_f32(PyObject* o, long long n, const char* what) { return static_cast<float*>(address(o, F32, n, what)); }
const int8_t* in_i8(PyObject* o, long long n, const char* what) { return static_cast<const int8_t*>(address(o, I8, n, what)); }
int8_t* out_i8(PyObject* o, long long n, const char* what) { return static_cast<int8_t*>(address(o, I8, n, what)); }
const int32_t* in_i32(PyObject* o, long long n, const char* what) { return static_cast<const int32_t*>(address(o, I32, n, what)); }

// The calls below hold no Python object while they run: other threads may go on, as with a ctypes call.
template <typename F>
glowmi_status without_gil(F f) {
  glowmi_status st;
  Py_BEGIN_ALLOW_THREADS
  st = f();
  Py_END_ALLOW_THREADS
  return st;
}

// A list of ("add", tensor[, QParam]) | ("mul", a) | ("max", a) | ("clip", a, b) as the library's op list.
struct Ops {
  glowmi_chain_op op[GLOWMI_MAX_CHAIN_OPS];
  int32_t n = 0;
  Ops(PyObject* list, at::ScalarType type, long long count) {
    PyObject* seq = PySequence_Fast(list, "ops: expected a list of op tuples");
    if (!seq) throw Refused{};
    try {
      fill(seq, type, count);
    } catch (...) {
      Py_DECREF(seq);
      throw;
    }
    Py_DECREF(seq);
  }

 private:
  void fill(PyObject* seq, at::ScalarType type, long long count) {
    const Py_ssize_t size = PySequence_Fast_GET_SIZE(seq);
    n = (int32_t)size;
    if (n > GLOWMI_MAX_CHAIN_OPS) return;                  // the library rejects the count before it reads an op
    for (int32_t i = 0; i < n; ++i) {
      PyObject* o = PySequence_Fast_GET_ITEM(seq, i);
      if (!PyTuple_Check(o) && !PyList_Check(o)) refuse(PyExc_TypeError, "ops: expected tuples");
      const Py_ssize_t len = PySequence_Fast_GET_SIZE(o);
      PyObject** item = PySequence_Fast_ITEMS(o);
      const char* kind = len > 0 && PyUnicode_Check(item[0]) ? PyUnicode_AsUTF8(item[0]) : "";
      if (!kind) throw Refused{};
      const std::string k(kind);
      auto need = [&](Py_ssize_t want) {
        if (len < want) refuse(PyExc_IndexError, "op " + std::to_string(i) + ": too few values");
      };
      glowmi_chain_op& c = op[i];
      c.a = c.b = 0.0f;
      c.tensor = nullptr;
      c.tensor_q = glowmi_qparam{1.0f, 0};
      if (k == "add") {
        need(2);
        c.kind = GLOWMI_OP_ADD_TENSOR;
        c.tensor = address(item[1], type, count, ("op " + std::to_string(i) + " tensor").c_str());
        if (len > 2) c.tensor_q = qparam_of(item[2]);
      } else if (k == "mul" || k == "max") {
        need(2);
        c.kind = k == "mul" ? GLOWMI_OP_MUL_SCALAR : GLOWMI_OP_MAX_SCALAR;
        c.a = number(item[1]);
      } else if (k == "clip") {
        need(3);
        c.kind = GLOWMI_OP_CLIP;
        c.a = number(item[1]);
        c.b = number(item[2]);
      } else {
        refuse(PyExc_ValueError, "unknown chain op '" + k + "'");
      }
    }
  }
};

// ---- the entry points: positional arguments as binding.py passes them; the calls without a shortcut tensor or
// planes are the general ones with None in their place --------------------------------------
int conv2d_packed(PyObject* const* a) {     // x, w, w_planes, bias, y, desc, addend, act, workspace, stream
  const Bytes ws = bytes_of(a[8], "workspace");
  View<glowmi_conv_desc> d(checked_desc(a[5]));
  const Counts c(*d.get());
  const Bytes planes = bytes_of(a[2], "planes", a[2] == Py_None ? 0 : glowmi_conv2d_filter_planes_bytes(d.get()));
  const glowmi_chain chain = {in_f32(a[6], c.y, "addend"), {1.0f, 0}, (glowmi_act)int32_of(a[7])};
  const float *x = in_f32(a[0], c.x, "x"), *w = in_f32(a[1], c.w, "w"), *b = in_f32(a[3], d.get()->k, "bias");
  float* y = out_f32(a[4], c.y, "y");
  const hipStream_t s = stream_of(a[9]);
  return without_gil([&] { return glowmi_conv2d_packed(x, w, planes.p, b, y, d.get(), &chain, ws.p, ws.n, s); });
}

int conv2d_pack_filter(PyObject* const* a) {   // w, desc, planes, stream
  View<glowmi_conv_desc> d(checked_desc(a[1]));
  const Counts c(*d.get());
  const Bytes planes = bytes_of(a[2], "planes");
  const float* w = in_f32(a[0], c.w, "w");
  const hipStream_t s = stream_of(a[3]);
  return without_gil([&] { return glowmi_conv2d_pack_filter(w, d.get(), planes.p, planes.n, s); });
}

int conv2d_chainv(PyObject* const* a) {     // x, w, bias, y, desc, ops, workspace, stream
  const Bytes ws = bytes_of(a[6], "workspace");
  View<glowmi_conv_desc> d(checked_desc(a[4]));
  const Counts c(*d.get());
  const Ops ops(a[5], F32, c.y);
  const float *x = in_f32(a[0], c.x, "x"), *w = in_f32(a[1], c.w, "w"), *b = in_f32(a[2], d.get()->k, "bias");
  float* y = out_f32(a[3], c.y, "y");
  const hipStream_t s = stream_of(a[7]);
  return without_gil([&] { return glowmi_conv2d_chainv(x, w, b, y, d.get(), ops.op, ops.n, ws.p, ws.n, s); });
}

int qconv2d_chain(PyObject* const* a) {     // x, xq, w, wq, bias, y, yq, desc, addend, addend_q, act, workspace, stream
  const Bytes ws = bytes_of(a[11], "workspace");
  View<glowmi_conv_desc> d(checked_desc(a[7]));
  const Counts c(*d.get());
  glowmi_chain chain = {in_i8(a[8], c.y, "addend"), {1.0f, 0}, (glowmi_act)int32_of(a[10])};
  if (a[9] != Py_None) chain.addend_q = qparam_of(a[9]);
  const int8_t *x = in_i8(a[0], c.x, "x"), *w = in_i8(a[2], c.w, "w");
  const int32_t* b = in_i32(a[4], d.get()->k, "bias");
  int8_t* y = out_i8(a[5], c.y, "y");
  const glowmi_qparam xq = qparam_of(a[1]), wq = qparam_of(a[3]), yq = qparam_of(a[6]);
  const hipStream_t s = stream_of(a[12]);
  return without_gil([&] { return glowmi_qconv2d_chain(x, xq, w, wq, b, y, yq, d.get(), &chain, ws.p, ws.n, s); });
}

int qconv2d_chainv(PyObject* const* a) {    // x, xq, w, wq, bias, y, yq, desc, ops, workspace, stream
  const Bytes ws = bytes_of(a[9], "workspace");
  View<glowmi_conv_desc> d(checked_desc(a[7]));
  const Counts c(*d.get());
  const Ops ops(a[8], I8, c.y);
  const int8_t *x = in_i8(a[0], c.x, "x"), *w = in_i8(a[2], c.w, "w");
  const int32_t* b = in_i32(a[4], d.get()->k, "bias");
  int8_t* y = out_i8(a[5], c.y, "y");
  const glowmi_qparam xq = qparam_of(a[1]), wq = qparam_of(a[3]), yq = qparam_of(a[6]);
  const hipStream_t s = stream_of(a[10]);
  return without_gil([&] { return glowmi_qconv2d_chainv(x, xq, w, wq, b, y, yq, d.get(), ops.op, ops.n, ws.p, ws.n, s); });
}

int fc_packed(PyObject* const* a) {         // a, w, w_planes, bias, y, M, K, N, act, workspace, stream
  const Bytes ws = bytes_of(a[9], "workspace");
  const int32_t M = extent(a[5], "M"), K = extent(a[6], "K"), N = extent(a[7], "N");
  const Bytes planes = bytes_of(a[2], "planes", a[2] == Py_None ? 0 : glowmi_fc_filter_planes_bytes(K, N));
  const float *x = in_f32(a[0], (long long)M * K, "a"), *w = in_f32(a[1], (long long)K * N, "w"), *b = in_f32(a[3], N, "bias");
  float* y = out_f32(a[4], (long long)M * N, "y");
  const glowmi_act act = (glowmi_act)int32_of(a[8]);
  const hipStream_t s = stream_of(a[10]);
  return without_gil([&] { return glowmi_fc_packed(x, w, planes.p, b, y, M, K, N, act, ws.p, ws.n, s); });
}

int fc_noalloc(PyObject* const* a) {        // a, w, bias, y, M, K, N, act, stream
  const int32_t M = extent(a[4], "M"), K = extent(a[5], "K"), N = extent(a[6], "N");
  const float *x = in_f32(a[0], (long long)M * K, "a"), *w = in_f32(a[1], (long long)K * N, "w"), *b = in_f32(a[2], N, "bias");
  float* y = out_f32(a[3], (long long)M * N, "y");
  const glowmi_act act = (glowmi_act)int32_of(a[7]);
  const hipStream_t s = stream_of(a[8]);
  return without_gil([&] { return glowmi_fc_noalloc(x, w, b, y, M, K, N, act, s); });
}

int fc_pack_filter(PyObject* const* a) {    // w, K, N, planes, stream
  const int32_t K = extent(a[1], "K"), N = extent(a[2], "N");
  const Bytes planes = bytes_of(a[3], "planes");
  const float* w = in_f32(a[0], (long long)K * N, "w");
  const hipStream_t s = stream_of(a[4]);
  return without_gil([&] { return glowmi_fc_pack_filter(w, K, N, planes.p, planes.n, s); });
}

int qfc(PyObject* const* a) {               // a, aq, w, wq, bias, y, yq, M, K, N, act, workspace, stream
  const Bytes ws = bytes_of(a[11], "workspace");
  const int32_t M = extent(a[7], "M"), K = extent(a[8], "K"), N = extent(a[9], "N");
  const int8_t *x = in_i8(a[0], (long long)M * K, "a"), *w = in_i8(a[2], (long long)K * N, "w");
  const int32_t* b = in_i32(a[4], N, "bias");
  int8_t* y = out_i8(a[5], (long long)M * N, "y");
  const glowmi_qparam xq = qparam_of(a[1]), wq = qparam_of(a[3]), yq = qparam_of(a[6]);
  const glowmi_act act = (glowmi_act)int32_of(a[10]);
  const hipStream_t s = stream_of(a[12]);
  return without_gil([&] { return glowmi_qfc(x, xq, w, wq, b, y, yq, M, K, N, act, ws.p, ws.n, s); });
}

int quantize(PyObject* const* a) {          // x, q, qp, count, stream
  const long long n = a[3] == Py_None ? tensor_of(a[0], "x").numel() : integer(a[3]);
  const float* x = in_f32(a[0], n, "x");
  int8_t* q = out_i8(a[1], n, "q");
  const glowmi_qparam qp = qparam_of(a[2]);
  const hipStream_t s = stream_of(a[4]);
  return without_gil([&] { return glowmi_quantize(x, q, (size_t)n, qp, s); });
}

int dequantize(PyObject* const* a) {        // q, x, qp, count, stream
  const long long n = a[3] == Py_None ? tensor_of(a[0], "q").numel() : integer(a[3]);
  const int8_t* q = in_i8(a[0], n, "q");
  float* x = out_f32(a[1], n, "x");
  const glowmi_qparam qp = qparam_of(a[2]);
  const hipStream_t s = stream_of(a[4]);
  return without_gil([&] { return glowmi_dequantize(q, x, (size_t)n, qp, s); });
}

int rescale(PyObject* const* a) {           // q_in, from_q, q_out, to_q, count, stream
  const long long n = a[4] == Py_None ? tensor_of(a[0], "q_in").numel() : integer(a[4]);
  const int8_t* in = in_i8(a[0], n, "q_in");
  int8_t* out = out_i8(a[2], n, "q_out");
  const glowmi_qparam from = qparam_of(a[1]), to = qparam_of(a[3]);
  const hipStream_t s = stream_of(a[5]);
  return without_gil([&] { return glowmi_rescale(in, from, out, to, (size_t)n, s); });
}

int seq_conv2d(PyObject* const* a) {        // x, layers, y, arena, stream
  const Bytes arena = bytes_of(a[3], "workspace");
  View<glowmi_seq_layer> l(checked_layers(a[1]));
  const Counts first(l.get()[0].desc), last(l.get()[l.count - 1].desc);
  const float* x = in_f32(a[0], first.x, "x");
  float* y = out_f32(a[2], last.y, "y");
  const hipStream_t s = stream_of(a[4]);
  return without_gil([&] { return glowmi_seq_conv2d(x, l.get(), (int32_t)l.count, y, arena.p, arena.n, s); });
}

int seq_qconv2d(PyObject* const* a) {       // x, xq, layers, y, arena, stream
  const Bytes arena = bytes_of(a[4], "workspace");
  View<glowmi_seq_layer> l(checked_layers(a[2]));
  const Counts first(l.get()[0].desc), last(l.get()[l.count - 1].desc);
  const int8_t* x = in_i8(a[0], first.x, "x");
  int8_t* y = out_i8(a[3], last.y, "y");
  const glowmi_qparam xq = qparam_of(a[1]);
  const hipStream_t s = stream_of(a[5]);
  return without_gil([&] { return glowmi_seq_qconv2d(x, xq, l.get(), (int32_t)l.count, y, arena.p, arena.n, s); });
}

// `address` for binding.py's own structures (layer lists): tensor, element type name, count, what it is.
PyObject* tensor_address(PyObject*, PyObject* const* a, Py_ssize_t n) {
  try {
    if (n != 4) refuse(PyExc_TypeError, "address takes 4 arguments");
    const char* type = PyUnicode_AsUTF8(a[1]);
    const char* what = PyUnicode_AsUTF8(a[3]);
    if (!type || !what) return nullptr;
    const std::string t(type);
    const at::ScalarType st = t == "int8" ? I8 : t == "int32" ? I32 : F32;
    void* p = address(a[0], st, a[2] == Py_None ? 0 : integer(a[2]), what);
    if (!p) Py_RETURN_NONE;
    return PyLong_FromVoidPtr(p);
  } catch (const Refused&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// Called once by binding.py: ConvDesc, QParam, SeqLayer.
PyObject* structure_types(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 3 || !PyType_Check(a[0]) || !PyType_Check(a[1]) || !PyType_Check(a[2])) {
    PyErr_SetString(PyExc_TypeError, "structure_types takes three classes");
    return nullptr;
  }
  PyObject** const held[3] = {&g_conv_desc, &g_qparam, &g_seq_layer};
  for (int i = 0; i < 3; ++i) {
    Py_INCREF(a[i]);
    Py_XSETREF(*held[i], a[i]);
  }
  Py_RETURN_NONE;
}

template <int (*F)(PyObject* const*), int N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  try {
    if (n != N) refuse(PyExc_TypeError, "wrong number of arguments");
    return PyLong_FromLong(F(args));
  } catch (const Refused&) {
    return nullptr;
  } catch (const std::exception& e) {      // torch's own errors (no stream without a GPU)
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

#define ENTRY(name, n) {#name, (PyCFunction)(void (*)(void))entry<name, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    ENTRY(conv2d_packed, 10), ENTRY(conv2d_pack_filter, 4), ENTRY(conv2d_chainv, 8),
    ENTRY(qconv2d_chain, 13), ENTRY(qconv2d_chainv, 11), ENTRY(fc_packed, 11), ENTRY(fc_noalloc, 9), ENTRY(fc_pack_filter, 5),
    ENTRY(qfc, 13), ENTRY(quantize, 5), ENTRY(dequantize, 5), ENTRY(rescale, 6), ENTRY(seq_conv2d, 5), ENTRY(seq_qconv2d, 6),
    {"structure_types", (PyCFunction)(void (*)(void))structure_types, METH_FASTCALL, nullptr},
    {"address", (PyCFunction)(void (*)(void))tensor_address, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Tensor-taking entry points of libglowmi.so.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
