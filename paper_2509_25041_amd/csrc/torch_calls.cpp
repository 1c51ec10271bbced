// The binding's calls that allocate their outputs, as a CPython module: allocations, checks and the library call without Python in
// between.  A planner's batch is three such calls with 18 tensors and 7 launches, and what the interpreter does for them (1.4 to 1.8 us a
// tensor, 2 to 3 us to marshal a call) was longer than the kernels: route, send lists and
// dispatch order of 16384 tokens 59.4 -> 41.8 us (kernels 39), of a single token 50.2 -> 30.8.
// Each function returns its tensors, or the library's status (an int) where that is not zero.
// The library's functions are handed over as addresses (bind), so that this module has one copy of it with ctypes.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/python_headers.h>

#include <ATen/ATen.h>

#include <algorithm>
#include <initializer_list>

#include "grace_moe.h"

namespace {

struct Library {
    decltype(&grace_workspace_bytes) workspace_bytes;
    decltype(&grace_route) route;
    decltype(&grace_permute) permute;
    decltype(&grace_route_permute) route_permute;
    decltype(&grace_send_lists_fresh) send_lists_fresh;
} lib = {};

// Releases the interpreter for the library call, as ctypes does.
template <typename F>
int call(F f) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

[[noreturn]] void refuse(PyObject *type, const char *text) {
    PyErr_SetString(type, text);
    throw python_error();
}
long integer(PyObject *o) {
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw python_error();
    return v;
}
template <typename T>
T *address(PyObject *o) {   // of the library's own object, or a stream
    void *p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw python_error();
    return (T *)p;
}
const at::Tensor &tensor(PyObject *o) {
    if (!THPVariable_Check(o)) refuse(PyExc_TypeError, "expected a tensor");
    return THPVariable_Unpack(o);
}
template <typename T>
T *data(const at::Tensor &t) {
    if (!t.is_cuda() || !t.is_contiguous()) refuse(PyExc_ValueError, "device tensors must be contiguous and live on the GPU");
    return (T *)t.data_ptr();
}
template <typename T>
T *data(PyObject *o) {
    return o == Py_None ? nullptr : data<T>(tensor(o));
}
grace_dtype dtype_code(const at::Tensor &t) {
    if (t.scalar_type() == at::kFloat) return GRACE_F32;
    if (t.scalar_type() == at::kBFloat16) return GRACE_BF16;
    refuse(PyExc_ValueError, "unsupported dtype");
}
void matrix(const at::Tensor &t, const char *what) {
    if (t.dim() != 2) refuse(PyExc_ValueError, what);
}
at::Tensor empty(at::IntArrayRef shape, at::ScalarType type, const at::Tensor &like) {
    return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}
PyObject *tuple(std::initializer_list<PyObject *> items) {   // takes the references
    PyObject *t = PyTuple_New((Py_ssize_t)items.size());
    Py_ssize_t i = 0;
    for (PyObject *o : items) {
        if (t) PyTuple_SET_ITEM(t, i++, o);
        else Py_XDECREF(o);
    }
    return t;
}
void expect(Py_ssize_t got, Py_ssize_t want) {
    if (!lib.route && want != 5) refuse(PyExc_RuntimeError, "the library has not been bound");
    if (got != want) refuse(PyExc_TypeError, "wrong number of arguments");
}

// bind(workspace_bytes, route, permute, route_permute, send_lists_fresh): addresses
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    expect(n, 5);
    lib = {(decltype(lib.workspace_bytes))address<void>(a[0]), (decltype(lib.route))address<void>(a[1]), (decltype(lib.permute))address<void>(a[2]),
           (decltype(lib.route_permute))address<void>(a[3]), (decltype(lib.send_lists_fresh))address<void>(a[4])};
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

struct Routed {
    at::Tensor expert, weight, inst, count;
    Routed(int64_t T, int64_t k, int64_t E, const at::Tensor &like)
        : expert(empty({T, k}, at::kInt, like)), weight(empty({T, k}, at::kFloat, like)), inst(empty({T, k}, at::kInt, like)),
          count(empty({E}, at::kInt, like)) {}
    PyObject *wrap() const { return tuple({THPVariable_Wrap(expert), THPVariable_Wrap(weight), THPVariable_Wrap(inst), THPVariable_Wrap(count)}); }
};
struct Permuted {
    at::Tensor pos, src, inst_off, rank_off, node_off, xp;
    Permuted(int64_t rows, int64_t I, int64_t R, int64_t N, const at::Tensor &like, const at::Tensor *x)
        : pos(empty({rows}, at::kInt, like)), src(empty({rows}, at::kInt, like)), inst_off(empty({I + 1}, at::kInt, like)),
          rank_off(empty({R + 1}, at::kInt, like)), node_off(empty({N + 1}, at::kInt, like)) {
        if (x) xp = empty({rows, x->size(1)}, x->scalar_type(), like);
    }
    PyObject *wrap() const {
        PyObject *rows = xp.defined() ? THPVariable_Wrap(xp) : (Py_INCREF(Py_None), Py_None);
        return tuple({THPVariable_Wrap(pos), THPVariable_Wrap(src), THPVariable_Wrap(inst_off), THPVariable_Wrap(rank_off),
                      THPVariable_Wrap(node_off), rows});
    }
};
at::Tensor workspace(int64_t T, int64_t E, int64_t k, int64_t I, const at::Tensor &like) {
    const size_t bytes = lib.workspace_bytes((int32_t)T, (int32_t)E, (int32_t)k, (int32_t)I, 0, 0, 0, GRACE_BF16);
    return empty({std::max<int64_t>((int64_t)bytes, 256)}, at::kByte, like);
}
// T and k as the library takes them
void sizes(int64_t T, int64_t k) {
    if (T > INT32_MAX || k > INT32_MAX || k < INT32_MIN) refuse(PyExc_ValueError, "sizes must fit 32 bits");
}

// route(table, I, local_rank, logits, k, renorm, rr_in, rr_out, policy, stream)
PyObject *route(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    expect(n, 10);
    const at::Tensor &logits = tensor(a[3]);
    matrix(logits, "logits must be [T, E]");
    if (logits.scalar_type() != at::kFloat) refuse(PyExc_ValueError, "logits must be float32");
    const int64_t T = logits.size(0), E = logits.size(1), k = integer(a[4]);
    sizes(T, k);
    const Routed r(T, k, E, logits);
    const at::Tensor ws = workspace(T, E, std::max<int64_t>(k, 1), integer(a[1]), logits);
    const auto *table = address<grace_table>(a[0]);
    const auto *lg = data<float>(logits);
    const auto *rr_in = data<uint32_t>(a[6]);
    auto *rr_out = data<uint32_t>(a[7]);
    const int local_rank = (int)integer(a[2]), renorm = (int)integer(a[5]), policy = (int)integer(a[8]);
    void *const stream = address<void>(a[9]);
    const int rc = call([&] {
        return lib.route(table, local_rank, (grace_policy)policy, lg, (int32_t)T, (int32_t)E, (int32_t)k, renorm, rr_in, rr_out,
                         data<int32_t>(r.expert), data<float>(r.weight), data<int32_t>(r.inst), data<int32_t>(r.count), data<void>(ws), stream);
    });
    return rc != GRACE_OK ? PyLong_FromLong(rc) : r.wrap();
    END_HANDLE_TH_ERRORS
}

// permute(table, E, I, R, N, topk_inst, x, stream)
PyObject *permute(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    expect(n, 8);
    const at::Tensor &inst = tensor(a[5]);
    matrix(inst, "topk_inst must be [T, k]");
    const at::Tensor *x = a[6] == Py_None ? nullptr : &tensor(a[6]);
    if (x) matrix(*x, "x must be [T, d]");
    const int64_t T = inst.size(0), k = inst.size(1), I = integer(a[2]);
    sizes(T, k);
    const grace_dtype dt = x ? dtype_code(*x) : GRACE_BF16;
    const int32_t d = x ? (int32_t)x->size(1) : 0;
    const Permuted p(T * k, I, integer(a[3]), integer(a[4]), inst, x);
    const at::Tensor ws = workspace(T, integer(a[1]), k, I, inst);
    const auto *table = address<grace_table>(a[0]);
    const auto *ti = data<int32_t>(inst);
    const void *const rows = x ? data<void>(*x) : nullptr;
    void *const stream = address<void>(a[7]);
    const int rc = call([&] {
        return lib.permute(table, ti, (int32_t)T, (int32_t)k, rows, d, dt, data<int32_t>(p.pos), data<int32_t>(p.src), data<int32_t>(p.inst_off),
                           data<int32_t>(p.rank_off), data<int32_t>(p.node_off), x ? data<void>(p.xp) : nullptr, data<void>(ws), stream);
    });
    return rc != GRACE_OK ? PyLong_FromLong(rc) : p.wrap();
    END_HANDLE_TH_ERRORS
}

// route_permute(table, I, R, N, local_rank, logits, k, x, renorm, rr_in, rr_out, policy, stream)
PyObject *route_permute(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    expect(n, 13);
    const at::Tensor &logits = tensor(a[5]);
    matrix(logits, "logits must be [T, E]");
    if (logits.scalar_type() != at::kFloat) refuse(PyExc_ValueError, "logits must be float32");
    const at::Tensor *x = a[7] == Py_None ? nullptr : &tensor(a[7]);
    if (x) matrix(*x, "x must be [T, d]");
    const int64_t T = logits.size(0), E = logits.size(1), k = integer(a[6]), I = integer(a[1]);
    sizes(T, k);
    const grace_dtype dt = x ? dtype_code(*x) : GRACE_BF16;
    const int32_t d = x ? (int32_t)x->size(1) : 0;
    const Routed r(T, k, E, logits);
    const Permuted p(T * k, I, integer(a[2]), integer(a[3]), logits, x);
    const at::Tensor ws = workspace(T, E, std::max<int64_t>(k, 1), I, logits);
    const auto *table = address<grace_table>(a[0]);
    const auto *lg = data<float>(logits);
    const void *const rows = x ? data<void>(*x) : nullptr;
    const auto *rr_in = data<uint32_t>(a[9]);
    auto *rr_out = data<uint32_t>(a[10]);
    const int local_rank = (int)integer(a[4]), renorm = (int)integer(a[8]), policy = (int)integer(a[11]);
    void *const stream = address<void>(a[12]);
    const int rc = call([&] {
        return lib.route_permute(table, local_rank, (grace_policy)policy, lg, (int32_t)T, (int32_t)E, (int32_t)k, renorm, rr_in, rr_out,
                                 data<int32_t>(r.expert), data<float>(r.weight), data<int32_t>(r.inst), data<int32_t>(r.count), rows, d, dt,
                                 data<int32_t>(p.pos), data<int32_t>(p.src), data<int32_t>(p.inst_off), data<int32_t>(p.rank_off),
                                 data<int32_t>(p.node_off), x ? data<void>(p.xp) : nullptr, data<void>(ws), stream);
    });
    if (rc != GRACE_OK) return PyLong_FromLong(rc);
    PyObject *const routed = r.wrap();
    return tuple({routed, p.wrap()});
    END_HANDLE_TH_ERRORS
}

// send_lists(table, E, I, R, N, local_rank, topk_inst, stream)
PyObject *send_lists(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    expect(n, 8);
    const at::Tensor &inst = tensor(a[6]);
    matrix(inst, "topk_inst must be [T, k]");
    const int64_t T = inst.size(0), k = inst.size(1), R = integer(a[3]), N = integer(a[4]);
    sizes(T, k);
    const at::Tensor rp = empty({R + 1}, at::kInt, inst), rt = empty({T * k}, at::kInt, inst), np = empty({N + 1}, at::kInt, inst),
                     nt = empty({T * k}, at::kInt, inst), ex = empty({T * k}, at::kInt, inst), tr = empty({4}, at::kLong, inst);
    const at::Tensor ws = workspace(T, integer(a[1]), k, integer(a[2]), inst);
    const auto *table = address<grace_table>(a[0]);
    const auto *ti = data<int32_t>(inst);
    const int local_rank = (int)integer(a[5]);
    void *const stream = address<void>(a[7]);
    const int rc = call([&] {
        return lib.send_lists_fresh(table, local_rank, ti, (int32_t)T, (int32_t)k, data<int32_t>(rp), data<int32_t>(rt), data<int32_t>(np),
                                    data<int32_t>(nt), data<int32_t>(ex), data<int64_t>(tr), data<void>(ws), stream);
    });
    if (rc != GRACE_OK) return PyLong_FromLong(rc);
    return tuple({THPVariable_Wrap(rp), THPVariable_Wrap(rt), THPVariable_Wrap(np), THPVariable_Wrap(nt), THPVariable_Wrap(ex), THPVariable_Wrap(tr)});
    END_HANDLE_TH_ERRORS
}

#define GRACE_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {GRACE_METHOD(bind), GRACE_METHOD(route), GRACE_METHOD(permute), GRACE_METHOD(route_permute), GRACE_METHOD(send_lists),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_calls(void) { return PyModule_Create(&module); }
