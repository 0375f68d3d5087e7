// The calls of binding.py that a program makes per step, from torch tensors to the C ABI without Python in between: outputs
// and scratch allocated, pointers taken and the launch made in one native call (a linear layer's host time 7.6 -> 5 us, of
// which two launches in flight are 4).
//
// Each function takes the plain case only - CUDA fp32 tensors of the layout that the call wants - and returns None for
// anything else, which binding.py then takes the long way, with that way's checks and errors.  A status other than 0 comes
// back as an int.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>

#include <algorithm>
#include <exception>

#include "lutnn.h"

namespace {

const lutnn_layer* layer_of(PyObject* address) { return static_cast<const lutnn_layer*>(PyLong_AsVoidPtr(address)); }
const lutnn_tree* tree_of(PyObject* address) { return static_cast<const lutnn_tree*>(PyLong_AsVoidPtr(address)); }

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// An ordinary CUDA tensor of fp32 with `dims` dimensions: no subclass, no transform's wrapper, no forward-mode tangent (which
// what the long way leaves to torch carries on).
bool plain(PyObject* object, int64_t dims) {
    if (!THPVariable_CheckExact(object) && Py_TYPE(object) != reinterpret_cast<PyTypeObject*>(ParameterClass)) return false;
    const at::Tensor& t = THPVariable_Unpack(object);
    static constexpr c10::DispatchKeySet kWrapped({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                                   c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Batched,
                                                   c10::DispatchKey::Functionalize, c10::DispatchKey::ZeroTensor,
                                                   c10::DispatchKey::Negative});
    return t.is_cuda() && t.scalar_type() == at::kFloat && t.dim() == dims && t.layout() == at::kStrided &&
           !t.key_set().has_any(kWrapped) && !t._fw_grad(0).defined();
}
bool rows(PyObject* object) { return plain(object, 2) && THPVariable_Unpack(object).stride(1) == 1; }
bool dense(PyObject* object, int64_t dims) { return plain(object, dims) && THPVariable_Unpack(object).is_contiguous(); }

at::Tensor empty(at::IntArrayRef shape, const at::Tensor& like, at::ScalarType type = at::kFloat) {
    return at::empty(shape, like.options().dtype(type).requires_grad(false));
}
float* data(const at::Tensor& t) { return t.defined() ? static_cast<float*>(t.data_ptr()) : nullptr; }
float* data(PyObject* object) { return data(THPVariable_Unpack(object)); }

PyObject* none() { Py_RETURN_NONE; }
PyObject* result(int status, const at::Tensor& out) { return status ? PyLong_FromLong(status) : THPVariable_Wrap(out); }

// Launches without the interpreter's lock, as ctypes does.  The call is one of the C ABI's on pointers taken before: a
// tensor's data may be refused with an exception, which must not leave here without the lock.
template <class Call>
int launch(Call&& call) {
    int status;
    Py_BEGIN_ALLOW_THREADS status = call();
    Py_END_ALLOW_THREADS return status;
}

// An exception (out of memory, a mode that gives no data pointers): the long way meets the same, and reports it.  One that
// came out of Python (a dispatch mode's) is still set there.
template <PyObject* (*Function)(PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject*, PyObject* const* args, Py_ssize_t n) {
    try {
        return Function(args, n);
    } catch (const std::exception&) {
        PyErr_Clear();
        return none();
    }
}

// linear(layer, X) and linear(layer, tree, X)
PyObject* linear(PyObject* const* args, Py_ssize_t n) {
    if ((n != 2 && n != 3) || !rows(args[n - 1])) return none();
    const lutnn_layer* layer = layer_of(args[0]);
    const lutnn_tree* tree = n == 3 ? tree_of(args[1]) : nullptr;
    const at::Tensor& X = THPVariable_Unpack(args[n - 1]);
    const int64_t N = X.size(0);
    const at::Tensor out = empty({N, layer->M}, X);
    const size_t bytes = lutnn_linear_scratch_bytes(layer, N, tree != nullptr);
    const at::Tensor scratch = bytes ? empty({(int64_t)bytes}, X, at::kByte) : at::Tensor();
    const int64_t ldx = X.stride(0), ldy = out.stride(0);
    float *x = data(X), *y = data(out), *w = data(scratch);
    void* s = stream();
    return result(launch([=] {
                      return tree ? lutnn_linear_tree_scratch(layer, tree, x, N, ldx, y, ldy, w, bytes, s)
                                  : lutnn_linear_scratch(layer, x, N, ldx, y, ldy, w, bytes, s);
                  }),
                  out);
}

PyObject* linear_tree16(PyObject* const* args, Py_ssize_t n) {
    if (n != 3 || !rows(args[2])) return none();
    const lutnn_layer* layer = layer_of(args[0]);
    const lutnn_tree* tree = tree_of(args[1]);
    const at::Tensor& X = THPVariable_Unpack(args[2]);
    const int64_t N = X.size(0);
    const at::Tensor out = empty({N, layer->M}, X), idx = empty({N, layer->C}, X, at::kShort);
    const int64_t ldx = X.stride(0), ldy = out.stride(0);
    float *x = data(X), *y = data(out);
    uint16_t* i = static_cast<uint16_t*>(idx.data_ptr());
    void* s = stream();
    return result(launch([=] { return lutnn_linear_tree16(layer, tree, x, N, ldx, y, ldy, i, s); }), out);
}

// Kernel, stride and padding as whole numbers.
bool square_geometry(const at::Tensor& inp, PyObject* const* args, lutnn_conv2d_geom* g) {
    int32_t v[3];
    for (int i = 0; i < 3; ++i) {
        if (!PyLong_CheckExact(args[i])) return false;
        int overflow = 0;
        const long x = PyLong_AsLongAndOverflow(args[i], &overflow);
        if (overflow || x < -(1 << 30) || x > (1 << 30)) return false;
        v[i] = (int32_t)x;
    }
    *g = {(int32_t)inp.size(1), (int32_t)inp.size(2), (int32_t)inp.size(3), v[0], v[0], v[1], v[1], v[2], v[2], 0};
    return true;
}

// conv2d(layer, inp, kernel, stride, pad)
PyObject* conv2d(PyObject* const* args, Py_ssize_t n) {
    if (n != 5 || !dense(args[1], 4)) return none();
    const lutnn_layer* layer = layer_of(args[0]);
    const at::Tensor& inp = THPVariable_Unpack(args[1]);
    lutnn_conv2d_geom g;
    if (!square_geometry(inp, args + 2, &g)) return none();
    const int64_t N = lutnn_conv2d_rows(&g, inp.size(0));
    if (N < 0) return none();
    const at::Tensor out = empty({N, layer->M}, inp);
    const size_t bytes = lutnn_conv2d_scratch_bytes(layer, N);
    const at::Tensor scratch = empty({(int64_t)bytes}, inp, at::kByte);
    const int64_t B = inp.size(0), ldy = out.stride(0);
    float *x = data(inp), *y = data(out), *w = data(scratch);
    void* s = stream();
    return result(launch([=, &g] { return lutnn_conv2d_scratch(layer, x, B, &g, y, ldy, w, bytes, s); }), out);
}

// build_table(centroids, W, dtype): (table, packed or None, scale or None)
PyObject* build_table(PyObject* const* args, Py_ssize_t n) {
    if (n != 3 || !dense(args[0], 3) || !rows(args[1]) || !PyLong_CheckExact(args[2])) return none();
    const at::Tensor &P = THPVariable_Unpack(args[0]), &W = THPVariable_Unpack(args[1]);
    const int64_t C = P.size(0), K = P.size(1), V = P.size(2), M = W.size(1);
    const long dtype = PyLong_AsLong(args[2]);
    if (W.size(0) != C * V || C > INT32_MAX || K > INT32_MAX || V > INT32_MAX || M > INT32_MAX) return none();
    at::Tensor table, packed, scale;
    if (dtype == LUTNN_TABLE_F32) {
        table = empty({C, K, M}, P);
    } else if (dtype == LUTNN_TABLE_I8 || dtype == LUTNN_TABLE_I4) {
        table = dtype == LUTNN_TABLE_I4 ? empty({C, K, (M + 1) / 2}, P, at::kByte) : empty({C, K, M}, P, at::kChar);
        scale = empty({1}, P);
        if (K <= 256)
            packed = empty({(int64_t)lutnn_packed_bytes((int32_t)C, (int32_t)K, (int32_t)M, (int32_t)dtype)}, P, at::kChar);
    } else {
        return none();
    }
    const int64_t ldw = W.stride(0);
    float *p = data(P), *w = data(W), *t = data(table), *pk = data(packed), *sc = data(scale);
    void* s = stream();
    const int status = launch([=] {
        return lutnn_build_table(p, w, ldw, (int32_t)C, (int32_t)K, (int32_t)V, (int32_t)M, (int32_t)dtype, t, pk, sc, s);
    });
    if (status) return PyLong_FromLong(status);
    return Py_BuildValue("NNN", THPVariable_Wrap(table), packed.defined() ? THPVariable_Wrap(packed) : none(),
                         scale.defined() ? THPVariable_Wrap(scale) : none());
}

// linear_gradient(G, W): Z, or False where another library's product is the one to take
PyObject* linear_gradient(PyObject* const* args, Py_ssize_t n) {
    if (n != 2 || !rows(args[0]) || !rows(args[1])) return none();
    const at::Tensor &G = THPVariable_Unpack(args[0]), &W = THPVariable_Unpack(args[1]);
    const int64_t N = G.size(0), D = W.size(0), M = W.size(1);
    if (G.size(1) != M || D > INT32_MAX || M > INT32_MAX) return none();
    const int64_t ldg = G.stride(0), ldw = W.stride(0);
    float *g = data(G), *w = data(W);
    if (!lutnn_linear_gradient_preferred(g, N, ldg, w, ldw, (int32_t)D, (int32_t)M)) Py_RETURN_FALSE;
    const at::Tensor Z = empty({N, D}, G);
    float* z = data(Z);
    void* s = stream();
    return result(launch([=] { return lutnn_linear_gradient(g, N, ldg, w, ldw, (int32_t)D, (int32_t)M, z, D, s); }), Z);
}

struct SoftPqOut {
    at::Tensor dP, dX, dt, workspace;
    SoftPqOut(int64_t C, int64_t K, int64_t V, int64_t N, const at::Tensor& X, bool need_dx) {
        dP = empty({C, K, V}, X);
        if (need_dx) dX = empty(X.sizes(), X);
        dt = empty({1}, X);
        const int64_t bytes = (int64_t)lutnn_softpq_workspace_bytes((int32_t)C, (int32_t)K, (int32_t)V, N);
        workspace = empty({std::max<int64_t>(bytes, 4)}, X, at::kByte);
    }
    PyObject* result(int status) const {
        if (status) return PyLong_FromLong(status);
        return Py_BuildValue("NNN", THPVariable_Wrap(dP), dX.defined() ? THPVariable_Wrap(dX) : none(), THPVariable_Wrap(dt));
    }
};

lutnn_layer shape_of(const at::Tensor& P, int64_t M) {
    lutnn_layer layer{};
    layer.C = (int32_t)P.size(0), layer.K = (int32_t)P.size(1), layer.V = (int32_t)P.size(2), layer.M = (int32_t)M;
    layer.table_dtype = LUTNN_TABLE_F32;
    layer.centroids = data(P);
    return layer;
}

// softpq_backward(centroids, M, temperature, X, Z, need_dx): (dP, dX or None, dt)
PyObject* softpq_backward(PyObject* const* args, Py_ssize_t n) {
    if (n != 6 || !dense(args[0], 3) || !rows(args[3]) || !rows(args[4])) return none();
    const at::Tensor &P = THPVariable_Unpack(args[0]), &X = THPVariable_Unpack(args[3]), &Z = THPVariable_Unpack(args[4]);
    if (X.sizes() != Z.sizes() || P.numel() > INT32_MAX || X.size(1) != P.size(0) * P.size(2)) return none();
    const lutnn_layer layer = shape_of(P, PyLong_AsLong(args[1]));
    const double t = PyFloat_AsDouble(args[2]);
    const SoftPqOut out(P.size(0), P.size(1), P.size(2), X.size(0), X, args[5] == Py_True);
    const int64_t N = X.size(0), ldx = X.stride(0), ldz = Z.stride(0), lddx = out.dX.defined() ? out.dX.stride(0) : 0;
    const int64_t bytes = out.workspace.numel();
    float *x = data(X), *z = data(Z), *dp = data(out.dP), *dx = data(out.dX), *dt = data(out.dt), *w = data(out.workspace);
    void* s = stream();
    return out.result(launch([=, &layer] {
        return lutnn_softpq_backward(&layer, (float)t, x, N, ldx, z, ldz, dp, dx, lddx, dt, w, bytes, s);
    }));
}

// softpq_backward_conv2d(centroids, temperature, inp, W, G, need_dx, kernel, stride, pad): (dP, dinp or None, dt)
PyObject* softpq_backward_conv2d(PyObject* const* args, Py_ssize_t n) {
    if (n != 9 || !dense(args[0], 3) || !dense(args[2], 4) || !rows(args[3]) || !dense(args[4], 4)) return none();
    const at::Tensor &P = THPVariable_Unpack(args[0]), &inp = THPVariable_Unpack(args[2]), &W = THPVariable_Unpack(args[3]),
                     &G = THPVariable_Unpack(args[4]);
    lutnn_conv2d_geom g;
    if (!square_geometry(inp, args + 6, &g) || P.numel() > INT32_MAX) return none();
    const int64_t N = lutnn_conv2d_rows(&g, inp.size(0)), D = P.size(0) * P.size(2), M = W.size(1);
    if (N < 0 || W.size(0) != D || M > INT32_MAX || G.numel() != N * M) return none();
    const lutnn_layer layer = shape_of(P, M);
    const double t = PyFloat_AsDouble(args[1]);
    const SoftPqOut out(P.size(0), P.size(1), P.size(2), N, inp, args[5] == Py_True);
    const at::Tensor Z = empty({N * D}, inp);
    const int64_t B = inp.size(0), ldw = W.stride(0), bytes = out.workspace.numel();
    float *x = data(inp), *w = data(W), *dy = data(G), *z = data(Z), *dp = data(out.dP), *dx = data(out.dX), *dt = data(out.dt);
    float* ws = data(out.workspace);
    void* s = stream();
    return out.result(launch([=, &layer, &g] {
        return lutnn_softpq_backward_conv2d(&layer, (float)t, x, B, &g, w, ldw, dy, z, dp, dx, dt, ws, bytes, s);
    }));
}

// bias_gradient(G): [N, M] or [B, M, Ho, Wo] summed over all but M
PyObject* bias_gradient(PyObject* const* args, Py_ssize_t n) {
    if (n != 1 || !(rows(args[0]) || dense(args[0], 4))) return none();
    const at::Tensor& G = THPVariable_Unpack(args[0]);
    const int64_t M = G.size(1), inner = G.dim() == 4 ? G.size(2) * G.size(3) : 1;
    // planes of one pixel are rows
    if (M < (inner == 1 ? 4 : 1) || M > INT32_MAX || inner < 1) return none();
    const at::Tensor out = empty({M}, G);
    const int64_t bytes = (int64_t)lutnn_bias_gradient_workspace_bytes(G.size(0), (int32_t)M, inner);
    const at::Tensor workspace = empty({std::max<int64_t>(bytes, 4)}, G, at::kByte);
    // the stride of a single row is whatever it is: a dimension of size 1 is contiguous with any
    const int64_t outer = G.size(0), ldg = outer > 1 ? G.stride(0) : M, size = workspace.numel();
    float *g = data(G), *y = data(out), *w = data(workspace);
    void* s = stream();
    return result(launch([=] { return lutnn_bias_gradient(g, outer, ldg, (int32_t)M, inner, y, w, size, s); }), out);
}

PyMethodDef kMethods[] = {
#define LUTNN_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(guarded<name>)), METH_FASTCALL, nullptr}
    LUTNN_METHOD(linear),          LUTNN_METHOD(linear_tree16),   LUTNN_METHOD(conv2d),
    LUTNN_METHOD(build_table),     LUTNN_METHOD(linear_gradient), LUTNN_METHOD(softpq_backward),
    LUTNN_METHOD(softpq_backward_conv2d), LUTNN_METHOD(bias_gradient), {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "torch_calls", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// Built from sources, and for a torch and an interpreter, of this hash: the loader can tell a stale file by it, as it does
// the library's.
extern "C" __attribute__((used, visibility("default"))) const char lutnn_torch_calls_version[] = "+" LUTNN_SOURCE_HASH;

PyMODINIT_FUNC PyInit_torch_calls() { return PyModule_Create(&kModule); }
