// Python argument marshalling of the device entry points of include/quamba_ssd.h, in native code.
//
// A generated token costs three library calls of 3 to 8 us of device work each at small batches, so what a call costs on
// the host is what a small model's token costs.  Marshalled in Python (about 50 attribute look-ups, tuple comparisons and
// ctypes conversions) a call took 8 to 11 us of host time; here the tensors' metadata are read from the tensor objects
// themselves.  Every check is made on every call; nothing is remembered from one call for the next but the
// addresses of the library's functions.
//
// The functions take positional arguments in the order of their Python signatures (binding.py) and return the library's
// status.  Tensors are torch tensors or None.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>

#include "quamba_ssd.h"

namespace {

// The library's entry points, by address: the library that binding.py has loaded.
struct Entry {
    decltype(&quamba_ssd_prefill_gated) prefill;
    decltype(&quamba_ssd_prefill_noalloc) prefill_noalloc;
    decltype(&quamba_ssd_decode_step_gated) decode;
    decltype(&quamba_ssd_decode_step_q8_gated) decode_q8;
    decltype(&quamba_ssd_quantize_state) quantize_state;
    decltype(&quamba_hadamard_quantize) hadamard;
    decltype(&quamba_mamba1_scan_gated) mamba1_scan;
    decltype(&quamba_mamba1_decode_step_gated) mamba1_decode;
    decltype(&quamba_conv1d_q8) conv1d;
} entry;

// The ctypes structures that carry the shape, the scale tables and the side inputs, and the classes that are read directly:
// types of binding.py.
PyObject *shape_type, *scales_type, *gate_struct_type, *device_scales_type, *gate_type;
PyObject *address_of;  // and its function from a ctypes pointer to its address or None

// Interned attribute names.
PyObject *s_tensors, *s_struct, *s_cuda_stream, *s_z, *s_z_scale, *s_dt_q, *s_dt_scale, *s_dt_bias;

struct Fail {};  // a Python exception is set

[[noreturn]] void fail(PyObject *type, const char *format, const char *name)
{
    PyErr_Format(type, format, name);
    throw Fail();
}

const at::Tensor *tensor_or_null(PyObject *o, const char *name)
{
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "%s must be a torch tensor", name);
    return &THPVariable_Unpack(o);
}

void *device_pointer(const at::Tensor *t, const char *name)
{
    if (!t) return nullptr;
    if (!t->is_cuda() || !t->is_contiguous()) fail(PyExc_ValueError, "%s must be a contiguous device tensor", name);
    return t->data_ptr();
}

// Device pointer of a tensor argument (None: NULL), with the checks a C caller would have to make itself.
template <typename T>
T *pointer(PyObject *o, at::ScalarType type, std::initializer_list<int64_t> shape, const char *name)
{
    const at::Tensor *t = tensor_or_null(o, name);
    if (!t) return nullptr;
    void *p = device_pointer(t, name);
    if (t->scalar_type() != type) {
        PyErr_Format(PyExc_ValueError, "%s must have dtype %s, got %s", name, c10::toString(type),
                     c10::toString(t->scalar_type()));
        throw Fail();
    }
    if (t->sizes() != at::IntArrayRef(shape)) {
        std::string want, got;
        for (int64_t v : shape) want += std::to_string(v) + ", ";
        for (int64_t v : t->sizes()) got += std::to_string(v) + ", ";
        PyErr_Format(PyExc_ValueError, "%s must have shape (%s), got (%s)", name, want.c_str(), got.c_str());
        throw Fail();
    }
    return static_cast<T *>(p);
}

float number(PyObject *o)
{
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Fail();
    return (float)v;
}

struct Ref {  // an owned reference
    PyObject *o;
    explicit Ref(PyObject *p) : o(p) { if (!o) throw Fail(); }
    ~Ref() { Py_DECREF(o); }
    Ref(const Ref &) = delete;
};

// The bytes of a ctypes structure, an instance of `type`: another object's bytes are not a structure, however many.
template <typename T>
T structure(PyObject *o, PyObject *type, const char *name)
{
    if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject *>(type))) {
        PyErr_Format(PyExc_TypeError, "%s must be a %s, not %s", name, reinterpret_cast<PyTypeObject *>(type)->tp_name,
                     Py_TYPE(o)->tp_name);
        throw Fail();
    }
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Fail();
    const bool fits = view.len >= (Py_ssize_t)sizeof(T);  // a subclass may have added fields
    T v;
    if (fits) memcpy(&v, view.buf, sizeof(T));
    PyBuffer_Release(&view);
    if (!fits) fail(PyExc_TypeError, "%s has the wrong size", name);
    return v;
}

quamba_ssd_shape_t shape_of(PyObject *o) { return structure<quamba_ssd_shape_t>(o, shape_type, "shape"); }

// The scale tables: a DeviceScales holds the five device tensors, in the struct's order; anything else (a subclass may say
// otherwise) is asked for its struct().
quamba_ssd_scales_t scales_of(PyObject *o)
{
    if (Py_TYPE(o) == reinterpret_cast<PyTypeObject *>(device_scales_type)) {
        Ref list(PyObject_GetAttr(o, s_tensors));
        if (PyList_Check(list.o) && PyList_GET_SIZE(list.o) == 5) {
            const void *p[5];
            int n = 0;
            for (; n < 5 && THPVariable_Check(PyList_GET_ITEM(list.o, n)); ++n)
                p[n] = THPVariable_Unpack(PyList_GET_ITEM(list.o, n)).data_ptr();
            if (n == 5)
                return {static_cast<const float *>(p[0]), static_cast<const int32_t *>(p[1]),
                        static_cast<const int32_t *>(p[2]), static_cast<const float *>(p[3]),
                        static_cast<const float *>(p[4])};
        }
    }
    Ref st(PyObject_CallMethodNoArgs(o, s_struct));
    return structure<quamba_ssd_scales_t>(st.o, scales_type, "scales.struct()");
}

PyObject *tuple_of(std::initializer_list<int64_t> v)
{
    PyObject *t = PyTuple_New((Py_ssize_t)v.size());
    Py_ssize_t i = 0;
    if (t)
        for (int64_t e : v) {
            PyObject *item = PyLong_FromLongLong(e);
            if (!item) {
                Py_DECREF(t);
                return nullptr;
            }
            PyTuple_SET_ITEM(t, i++, item);
        }
    return t;
}

// The optional side inputs (None: no struct): the fields of a Gate; anything else is asked for its struct().
struct GateArg {
    quamba_ssd_gate_t g;
    bool present = false;
    GateArg(PyObject *o, std::initializer_list<int64_t> z_shape, std::initializer_list<int64_t> dt_shape, int64_t nbias)
    {
        if (o == Py_None) return;
        present = true;
        if (Py_TYPE(o) != reinterpret_cast<PyTypeObject *>(gate_type)) {
            Ref zt(tuple_of(z_shape)), dtt(tuple_of(dt_shape)), nb(PyLong_FromLongLong(nbias));
            Ref st(PyObject_CallMethodObjArgs(o, s_struct, zt.o, dtt.o, nb.o, nullptr));
            g = structure<quamba_ssd_gate_t>(st.o, gate_struct_type, "gate.struct()");
            return;
        }
        Ref z(PyObject_GetAttr(o, s_z)), zs(PyObject_GetAttr(o, s_z_scale)), dq(PyObject_GetAttr(o, s_dt_q)),
            ds(PyObject_GetAttr(o, s_dt_scale)), db(PyObject_GetAttr(o, s_dt_bias));
        g.z = pointer<int8_t>(z.o, at::kChar, z_shape, "gate.z");
        g.z_scale = number(zs.o);
        g.dt_q = pointer<int8_t>(dq.o, at::kChar, dt_shape, "gate.dt_q");
        g.dt_scale = number(ds.o);
        g.dt_bias = pointer<float>(db.o, at::kFloat, {nbias}, "gate.dt_bias");
    }
    const quamba_ssd_gate_t *get() const { return present ? &g : nullptr; }
};

// The stream argument: None is torch's current stream, else an object with a cuda_stream attribute or the pointer itself, as
// a number or as anything that ctypes takes for a pointer (c_void_p, a pointer or array instance).
void *stream_of(PyObject *o)
{
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    PyObject *a = PyObject_GetAttr(o, s_cuda_stream);
    if (!a) {
        PyErr_Clear();
        Py_INCREF(o);
        a = o;
    }
    Ref held(a);
    if (!PyLong_Check(a)) {
        Ref address(PyObject_CallFunctionObjArgs(address_of, a, nullptr));
        if (address.o == Py_None) return nullptr;
        void *p = PyLong_AsVoidPtr(address.o);
        if (PyErr_Occurred()) throw Fail();
        return p;
    }
    void *p = PyLong_AsVoidPtr(a);
    if (PyErr_Occurred()) throw Fail();
    return p;
}

void need(Py_ssize_t n, Py_ssize_t want)
{
    if (n != want) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
        throw Fail();
    }
}

// Runs a library call without the interpreter lock and hands its status back.
template <typename F>
PyObject *call(F &&f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// Arguments of the SSD entry points that prefill and decode share.
struct Operands {
    const int8_t *x, *B, *C;
    const float *dt, *A, *D;
};

Operands prefill_operands(PyObject *const *a, const quamba_ssd_shape_t &s)
{
    Operands o;
    o.x = pointer<int8_t>(a[0], at::kChar, {s.batch, s.seqlen, s.nheads, s.headdim}, "x");
    o.B = pointer<int8_t>(a[1], at::kChar, {s.batch, s.seqlen, s.ngroups, s.d_state}, "B");
    o.C = pointer<int8_t>(a[2], at::kChar, {s.batch, s.seqlen, s.ngroups, s.d_state}, "C");
    o.dt = pointer<float>(a[3], at::kFloat, {s.batch, s.seqlen, s.nheads}, "dt");
    o.A = pointer<float>(a[4], at::kFloat, {s.nheads}, "A");
    o.D = pointer<float>(a[5], at::kFloat, {s.nheads}, "D");
    return o;
}

Operands decode_operands(PyObject *const *a, const quamba_ssd_shape_t &s)
{
    Operands o;
    o.x = pointer<int8_t>(a[0], at::kChar, {s.batch, s.nheads, s.headdim}, "x");
    o.B = pointer<int8_t>(a[1], at::kChar, {s.batch, s.ngroups, s.d_state}, "B");
    o.C = pointer<int8_t>(a[2], at::kChar, {s.batch, s.ngroups, s.d_state}, "C");
    o.dt = pointer<float>(a[3], at::kFloat, {s.batch, s.nheads}, "dt");
    o.A = pointer<float>(a[4], at::kFloat, {s.nheads}, "A");
    o.D = pointer<float>(a[5], at::kFloat, {s.nheads}, "D");
    return o;
}

// shape, scales, x, B, C, dt, A, D, init_state, y, final_state, workspace, stream, gate
PyObject *prefill(PyObject *const *a)
{
    const quamba_ssd_shape_t s = shape_of(a[0]);
    const quamba_ssd_scales_t sc = scales_of(a[1]);
    const at::Tensor *w = tensor_or_null(a[11], "workspace");
    void *ws = device_pointer(w, "workspace");
    const size_t ws_bytes = w ? (size_t)w->numel() * w->element_size() : 0;
    const GateArg gate(a[13], {s.batch, s.seqlen, s.nheads, s.headdim}, {s.batch, s.seqlen, s.nheads}, s.nheads);
    const Operands o = prefill_operands(a + 2, s);
    const float *init = pointer<float>(a[8], at::kFloat, {s.batch, s.nheads, s.headdim, s.d_state}, "init_state");
    uint16_t *y = pointer<uint16_t>(a[9], at::kHalf, {s.batch, s.seqlen, s.nheads, s.headdim}, "y");
    float *fin = pointer<float>(a[10], at::kFloat, {s.batch, s.nheads, s.headdim, s.d_state}, "final_state");
    void *stream = stream_of(a[12]);
    return call([&] {
        return entry.prefill(&s, &sc, gate.get(), o.x, o.B, o.C, o.dt, o.A, o.D, init, y, fin, ws, ws_bytes, stream);
    });
}

// shape, scales, x, B, C, dt, A, D, init_state, y, final_state, stream
PyObject *prefill_noalloc(PyObject *const *a)
{
    const quamba_ssd_shape_t s = shape_of(a[0]);
    const quamba_ssd_scales_t sc = scales_of(a[1]);
    const Operands o = prefill_operands(a + 2, s);
    const float *init = pointer<float>(a[8], at::kFloat, {s.batch, s.nheads, s.headdim, s.d_state}, "init_state");
    uint16_t *y = pointer<uint16_t>(a[9], at::kHalf, {s.batch, s.seqlen, s.nheads, s.headdim}, "y");
    float *fin = pointer<float>(a[10], at::kFloat, {s.batch, s.nheads, s.headdim, s.d_state}, "final_state");
    void *stream = stream_of(a[11]);
    return call([&] {
        return entry.prefill_noalloc(&s, &sc, o.x, o.B, o.C, o.dt, o.A, o.D, init, y, fin, stream);
    });
}

// shape, scales, x, B, C, dt, A, D, state, y, stream, gate
PyObject *decode(PyObject *const *a)
{
    const quamba_ssd_shape_t s = shape_of(a[0]);
    const quamba_ssd_scales_t sc = scales_of(a[1]);
    const GateArg gate(a[11], {s.batch, s.nheads, s.headdim}, {s.batch, s.nheads}, s.nheads);
    const Operands o = decode_operands(a + 2, s);
    float *state = pointer<float>(a[8], at::kFloat, {s.batch, s.nheads, s.headdim, s.d_state}, "state");
    uint16_t *y = pointer<uint16_t>(a[9], at::kHalf, {s.batch, s.nheads, s.headdim}, "y");
    void *stream = stream_of(a[10]);
    return call([&] { return entry.decode(&s, &sc, gate.get(), o.x, o.B, o.C, o.dt, o.A, o.D, state, y, stream); });
}

int64_t cells(const quamba_ssd_shape_t &s) { return (int64_t)s.ngroups * s.n_head_clusters * s.n_chan_clusters; }

// shape, scales, state_scales, x, B, C, dt, A, D, state_q, y, stream, gate
PyObject *decode_q8(PyObject *const *a)
{
    const quamba_ssd_shape_t s = shape_of(a[0]);
    const quamba_ssd_scales_t sc = scales_of(a[1]);
    const GateArg gate(a[12], {s.batch, s.nheads, s.headdim}, {s.batch, s.nheads}, s.nheads);
    const float *ss = pointer<float>(a[2], at::kFloat, {cells(s), s.d_state}, "state_scales");
    const Operands o = decode_operands(a + 3, s);
    int8_t *state = pointer<int8_t>(a[9], at::kChar, {s.batch, s.nheads, s.headdim, s.d_state}, "state_q");
    uint16_t *y = pointer<uint16_t>(a[10], at::kHalf, {s.batch, s.nheads, s.headdim}, "y");
    void *stream = stream_of(a[11]);
    return call([&] {
        return entry.decode_q8(&s, &sc, gate.get(), ss, o.x, o.B, o.C, o.dt, o.A, o.D, state, y, stream);
    });
}

// shape, scales, state_scales, state, state_q, stream
PyObject *quantize_state(PyObject *const *a)
{
    const quamba_ssd_shape_t s = shape_of(a[0]);
    const quamba_ssd_scales_t sc = scales_of(a[1]);
    const float *ss = pointer<float>(a[2], at::kFloat, {cells(s), s.d_state}, "state_scales");
    const float *state = pointer<float>(a[3], at::kFloat, {s.batch, s.nheads, s.headdim, s.d_state}, "state");
    int8_t *q = pointer<int8_t>(a[4], at::kChar, {s.batch, s.nheads, s.headdim, s.d_state}, "state_q");
    void *stream = stream_of(a[5]);
    return call([&] { return entry.quantize_state(&s, &sc, ss, state, q, stream); });
}

// y, s_y, out, stream
PyObject *hadamard(PyObject *const *a)
{
    const at::Tensor *y = tensor_or_null(a[0], "y");
    if (!y || y->dim() == 0) fail(PyExc_ValueError, "%s must be a tensor of rows", "y");
    const int64_t n = y->size(-1), rows = y->numel() / (n > 1 ? n : 1);
    if (rows == 0 && n > 0) return PyLong_FromLong(QUAMBA_OK);  // an empty tensor has no device pointer to pass
    const float s_y = number(a[1]);
    void *yp = device_pointer(y, "y");
    if (y->scalar_type() != at::kHalf) fail(PyExc_ValueError, "%s must have dtype torch.float16", "y");
    const at::Tensor *out = tensor_or_null(a[2], "out");
    void *op = device_pointer(out, "out");
    if (out && out->scalar_type() != at::kChar) fail(PyExc_ValueError, "%s must have dtype torch.int8", "out");
    if (out && out->sizes() != y->sizes()) fail(PyExc_ValueError, "%s must have the shape of y", "out");
    void *stream = stream_of(a[3]);
    return call([&] {
        return entry.hadamard(static_cast<const uint16_t *>(yp), rows, n > INT32_MAX ? 0 : (int32_t)n, s_y,
                              static_cast<int8_t *>(op), stream);
    });
}

// shape, scales, x, B, C, dt, A, D, y, init_state, final_state, stream, gate
PyObject *mamba1_scan(PyObject *const *a)
{
    const quamba_ssd_shape_t s = shape_of(a[0]);
    const quamba_ssd_scales_t sc = scales_of(a[1]);
    const int64_t b = s.batch, L = s.seqlen, D = s.headdim, N = s.d_state;
    const int8_t *x = pointer<int8_t>(a[2], at::kChar, {b, D, L}, "x");
    const int8_t *B = pointer<int8_t>(a[3], at::kChar, {b, N, L}, "B");
    const int8_t *C = pointer<int8_t>(a[4], at::kChar, {b, N, L}, "C");
    const float *dt = pointer<float>(a[5], at::kFloat, {b, D, L}, "dt");
    const float *A = pointer<float>(a[6], at::kFloat, {D, N}, "A");
    const float *Dk = pointer<float>(a[7], at::kFloat, {D}, "D");
    const float *init = pointer<float>(a[9], at::kFloat, {b, D, N}, "init_state");
    uint16_t *y = pointer<uint16_t>(a[8], at::kHalf, {b, D, L}, "y");
    float *fin = pointer<float>(a[10], at::kFloat, {b, D, N}, "final_state");
    void *stream = stream_of(a[11]);
    const GateArg gate(a[12], {b, D, L}, {b, D, L}, D);
    return call([&] { return entry.mamba1_scan(&s, &sc, gate.get(), x, B, C, dt, A, Dk, init, y, fin, stream); });
}

// shape, scales, x, B, C, dt, A, D, state, y, stream, gate
PyObject *mamba1_decode(PyObject *const *a)
{
    const quamba_ssd_shape_t s = shape_of(a[0]);
    const quamba_ssd_scales_t sc = scales_of(a[1]);
    const int64_t b = s.batch, D = s.headdim, N = s.d_state;
    const int8_t *x = pointer<int8_t>(a[2], at::kChar, {b, D}, "x");
    const int8_t *B = pointer<int8_t>(a[3], at::kChar, {b, N}, "B");
    const int8_t *C = pointer<int8_t>(a[4], at::kChar, {b, N}, "C");
    const float *dt = pointer<float>(a[5], at::kFloat, {b, D}, "dt");
    const float *A = pointer<float>(a[6], at::kFloat, {D, N}, "A");
    const float *Dk = pointer<float>(a[7], at::kFloat, {D}, "D");
    float *state = pointer<float>(a[8], at::kFloat, {b, D, N}, "state");
    uint16_t *y = pointer<uint16_t>(a[9], at::kHalf, {b, D}, "y");
    void *stream = stream_of(a[10]);
    const GateArg gate(a[11], {b, D}, {b, D}, D);
    return call([&] { return entry.mamba1_decode(&s, &sc, gate.get(), x, B, C, dt, A, Dk, state, y, stream); });
}

// shape, scales, xBC, weight, bias, in_w_scale, x_out, B_out, C_out, conv_state_in, conv_state_out, stream
PyObject *conv1d(PyObject *const *a)
{
    const quamba_ssd_shape_t s = shape_of(a[0]);
    const quamba_ssd_scales_t sc = scales_of(a[1]);
    const int64_t b = s.batch, L = s.seqlen, H = s.nheads, P = s.headdim, G = s.ngroups, N = s.d_state;
    const int64_t Ct = H * P + 2 * G * N;
    const int8_t *in = pointer<int8_t>(a[2], at::kChar, {b, L, Ct}, "xBC");
    const int8_t *weight = pointer<int8_t>(a[3], at::kChar, {Ct, 4}, "weight");
    const float *bias = pointer<float>(a[4], at::kFloat, {Ct}, "bias");
    const float scale = number(a[5]);
    const int8_t *st_in = pointer<int8_t>(a[9], at::kChar, {b, 3, Ct}, "conv_state_in");
    int8_t *x = pointer<int8_t>(a[6], at::kChar, {b, L, H, P}, "x_out");
    int8_t *B = pointer<int8_t>(a[7], at::kChar, {b, L, G, N}, "B_out");
    int8_t *C = pointer<int8_t>(a[8], at::kChar, {b, L, G, N}, "C_out");
    int8_t *st_out = pointer<int8_t>(a[10], at::kChar, {b, 3, Ct}, "conv_state_out");
    void *stream = stream_of(a[11]);
    return call([&] { return entry.conv1d(&s, &sc, in, weight, bias, scale, st_in, x, B, C, st_out, stream); });
}

template <PyObject *(*F)(PyObject *const *), int N>
PyObject *method(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    try {
        need(n, N);
        return F(a);
    } catch (const Fail &) {
        return nullptr;
    } catch (const std::exception &e) {  // torch's own errors (a tensor without storage, a lost device)
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// The addresses of the library's functions, in the order of Entry, and what binding.py has for the objects above.
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    constexpr int kEntries = 9;
    PyObject **const objects[] = {&shape_type, &scales_type, &gate_struct_type, &device_scales_type, &gate_type, &address_of};
    constexpr int kObjects = sizeof(objects) / sizeof(objects[0]);
    void *p[kEntries];
    if (n != kEntries + kObjects) {
        PyErr_Format(PyExc_TypeError, "expected %d addresses and %d objects", kEntries, kObjects);
        return nullptr;
    }
    for (int i = 0; i < kEntries; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    for (int i = 0; i < kObjects; ++i) {
        if (i + 1 < kObjects ? !PyType_Check(a[kEntries + i]) : !PyCallable_Check(a[kEntries + i])) {
            PyErr_SetString(PyExc_TypeError, "expected types and a function");
            return nullptr;
        }
        Py_INCREF(a[kEntries + i]);
        Py_XDECREF(*objects[i]);
        *objects[i] = a[kEntries + i];
    }
    static_assert(sizeof(Entry) == sizeof(p), "one address per entry point");
    memcpy(&entry, p, sizeof(entry));
    Py_RETURN_NONE;
}

#define QUAMBA_METHOD(name, nargs) \
    {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&method<name, nargs>)), METH_FASTCALL, nullptr}

PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&bind)), METH_FASTCALL, nullptr},
    QUAMBA_METHOD(prefill, 14),
    QUAMBA_METHOD(prefill_noalloc, 12),
    QUAMBA_METHOD(decode, 12),
    QUAMBA_METHOD(decode_q8, 13),
    QUAMBA_METHOD(quantize_state, 6),
    QUAMBA_METHOD(hadamard, 4),
    QUAMBA_METHOD(mamba1_scan, 13),
    QUAMBA_METHOD(mamba1_decode, 12),
    QUAMBA_METHOD(conv1d, 12),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bind(void)
{
    const struct { PyObject **to; const char *text; } names[] = {
        {&s_tensors, "tensors"}, {&s_struct, "struct"}, {&s_cuda_stream, "cuda_stream"}, {&s_z, "z"},
        {&s_z_scale, "z_scale"}, {&s_dt_q, "dt_q"}, {&s_dt_scale, "dt_scale"}, {&s_dt_bias, "dt_bias"}};
    for (const auto &e : names)
        if (!(*e.to = PyUnicode_InternFromString(e.text))) return nullptr;
    return PyModule_Create(&module);
}
