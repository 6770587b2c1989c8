// host.cpp -- the per-step calls of include/picasso.h for Python: a CPython module that checks tensors, allocates
// outputs (with torch's allocator, on the current stream) and calls the library.  Through ctypes a call took about 12
// microseconds of Python, several times what its kernel runs on a small mesh; through this module about 5.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "../../include/picasso.h"

namespace {

PyObject* g_current_device = nullptr;  // () -> index of the current device
PyObject* g_current_stream = nullptr;  // (device index) -> its current stream as a number
PyObject* g_raise = nullptr;           // (context, status): raises the exception for a failed call

struct PyError {};  // a Python exception has been set

[[noreturn]] void fail(PyObject* type, const char* text) {
    PyErr_SetString(type, text);
    throw PyError{};
}

// The positional arguments of a call.
struct Args {
    PyObject* const* a;
    Py_ssize_t n, at = 0;
    PyObject* next() {
        if (at >= n) fail(PyExc_TypeError, "too few arguments");
        return a[at++];
    }
    long long integer() {
        PyObject* o = next();
        long long v;
        if (PyLong_Check(o)) {
            v = PyLong_AsLongLong(o);
        } else {
            PyObject* l = PyNumber_Long(o);
            if (!l) throw PyError{};
            v = PyLong_AsLongLong(l);
            Py_DECREF(l);
        }
        if (v == -1 && PyErr_Occurred()) throw PyError{};
        return v;
    }
    int i32() { return (int)integer(); }
    picasso_ctx* context() { return reinterpret_cast<picasso_ctx*>((intptr_t)integer()); }
    void* stream() {
        PyObject* o = next();
        PyObject* number;
        if (o == Py_None) {
            PyObject* device = PyObject_CallNoArgs(g_current_device);
            if (!device) throw PyError{};
            number = PyObject_CallOneArg(g_current_stream, device);
            Py_DECREF(device);
        } else {
            number = PyObject_GetAttrString(o, "cuda_stream");
        }
        if (!number) throw PyError{};
        void* s = PyLong_AsVoidPtr(number);
        Py_DECREF(number);
        if (PyErr_Occurred()) throw PyError{};
        return s;
    }
    // a contiguous CUDA tensor of the given type, or (unless its shape is needed) null for None
    const at::Tensor* tensor(at::ScalarType type, const char* what, bool required) {
        PyObject* o = next();
        if (o == Py_None && !required) return nullptr;
        if (THPVariable_Check(o)) {
            const at::Tensor& t = THPVariable_Unpack(o);
            if (t.is_cuda() && t.scalar_type() == type && t.is_contiguous()) return &t;
        }
        PyObject* shape = required ? PyObject_GetAttrString(o, "shape") : nullptr;
        if (required && !shape) throw PyError{};  // (not an array at all)
        Py_XDECREF(shape);
        PyErr_Format(PyExc_TypeError, "%s: expected a contiguous CUDA tensor of dtype %s", what,
                     type == at::kFloat ? "torch.float32" : "torch.int32");
        throw PyError{};
    }
    const at::Tensor& f32(const char* what) { return *tensor(at::kFloat, what, true); }
    const at::Tensor& ints(const char* what) { return *tensor(at::kInt, what, true); }
    const at::Tensor* maybe_f32(const char* what) { return tensor(at::kFloat, what, false); }
    const at::Tensor* maybe_ints(const char* what) { return tensor(at::kInt, what, false); }
};

int rows(const at::Tensor& t, int dim = 0) {
    if (t.dim() <= dim) fail(PyExc_IndexError, "tuple index out of range");
    return (int)t.size(dim);
}
at::Tensor out_f32(at::IntArrayRef shape, const at::Tensor& like) { return at::empty(shape, at::TensorOptions().dtype(at::kFloat).device(like.device())); }
at::Tensor out_i32(at::IntArrayRef shape, const at::Tensor& like) { return at::empty(shape, at::TensorOptions().dtype(at::kInt).device(like.device())); }
float* F(const at::Tensor& t) { return static_cast<float*>(t.data_ptr()); }
int32_t* I(const at::Tensor& t) { return static_cast<int32_t*>(t.data_ptr()); }
float* F(const at::Tensor* t) { return t ? F(*t) : nullptr; }
int32_t* I(const at::Tensor* t) { return t ? I(*t) : nullptr; }

// The library's call without the interpreter's lock.
template <class Call>
int unlocked(Call call) {
    PyThreadState* s = PyEval_SaveThread();
    const int st = call();
    PyEval_RestoreThread(s);
    return st;
}
template <class Call>
void checked(picasso_ctx* c, Call call) {
    const int st = unlocked(call);
    if (st == PICASSO_OK) return;
    PyObject* r = PyObject_CallFunction(g_raise, "Ki", (unsigned long long)(intptr_t)c, st);
    Py_XDECREF(r);
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "a library call failed");
    throw PyError{};
}

PyObject* wrap(at::Tensor t) { return THPVariable_Wrap(std::move(t)); }
PyObject* pack(std::initializer_list<PyObject*> items) {
    PyObject* t = PyTuple_New((Py_ssize_t)items.size());
    Py_ssize_t i = 0;
    for (PyObject* o : items) PyTuple_SET_ITEM(t, i++, o);
    return t;
}
PyObject* none() { Py_RETURN_NONE; }

// Exceptions of C++ become Python's, torch's (an allocation that fails, say) the ones that torch raises for them.
template <PyObject* (*Body)(Args&)>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n) {
    try {
        Args args{a, n};
        return Body(args);
    } catch (const PyError&) {
    } catch (...) {
        torch::translate_exception_to_python(std::current_exception());
    }
    return nullptr;
}

PyObject* decimate(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor &v = a.f32("verts"), &f = a.ints("facets");
    const int target = a.i32();
    const at::Tensor *vo_ = a.maybe_f32("verts_out"), *fo_ = a.maybe_ints("facets_out"), *cid_ = a.maybe_ints("cluster_id");
    picasso_stats* stats = reinterpret_cast<picasso_stats*>((intptr_t)a.integer());
    const int N = rows(v), nF = rows(f);
    const at::Tensor vo = vo_ ? *vo_ : out_f32({std::max(N, 1), 3}, v), fo = fo_ ? *fo_ : out_i32({std::max(nF, 1), 3}, v),
                     cid = cid_ ? *cid_ : out_i32({std::max(N, 1)}, v);
    int32_t nv = 0, nf = 0;
    const int st = unlocked([&] { return picasso_decimate(c, s, F(v), N, I(f), nF, target, F(vo), I(fo), I(cid), &nv, &nf, stats); });
    if (st < 0) return pack({PyLong_FromLong(st), none(), none(), none()});
    return pack({PyLong_FromLong(st), wrap(vo.narrow(0, 0, nv)), wrap(fo.narrow(0, 0, nf)), wrap(cid.narrow(0, 0, N))});
}

// n int32 values of an object with the buffer interface (a contiguous numpy array)
struct HostInts {
    Py_buffer b{};
    HostInts(PyObject* o, bool writable) {
        if (PyObject_GetBuffer(o, &b, writable ? PyBUF_CONTIG : PyBUF_CONTIG_RO) != 0) throw PyError{};
    }
    ~HostInts() { PyBuffer_Release(&b); }
    HostInts(const HostInts&) = delete;
    int n() const { return (int)(b.len / 4); }
    int32_t* p() const { return static_cast<int32_t*>(b.buf); }
};

PyObject* decimate_batch(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor &v = a.f32("verts"), &f = a.ints("facets");
    const HostInts nv_in(a.next(), false), nf_in(a.next(), false), target(a.next(), false);
    const at::Tensor *vo_ = a.maybe_f32("verts_out"), *fo_ = a.maybe_ints("facets_out"), *cid_ = a.maybe_ints("cluster_id");
    const HostInts nv_out(a.next(), true), nf_out(a.next(), true);
    picasso_stats* stats = reinterpret_cast<picasso_stats*>((intptr_t)a.integer());
    const int N = rows(v), nF = rows(f), B = nv_in.n();
    if (nf_in.n() < B || target.n() < B || nv_out.n() < B || nf_out.n() < B) fail(PyExc_ValueError, "nv_in, nf_in and target_nv differ in length");
    const at::Tensor vo = vo_ ? *vo_ : out_f32({std::max(N, 1), 3}, v), fo = fo_ ? *fo_ : out_i32({std::max(nF, 1), 3}, v),
                     cid = cid_ ? *cid_ : out_i32({std::max(N, 1)}, v);
    const int st = unlocked([&] {
        return picasso_decimate_batch(c, s, B, F(v), I(f), nv_in.p(), nf_in.p(), target.p(), F(vo), I(fo), I(cid), nv_out.p(),
                                      nf_out.p(), stats);
    });
    if (st < 0) return pack({PyLong_FromLong(st), none(), none(), none()});
    long long nv = 0, nf = 0;
    for (int b = 0; b < B; ++b) {
        nv += nv_out.p()[b];
        nf += nf_out.p()[b];
    }
    return pack({PyLong_FromLong(st), wrap(vo.narrow(0, 0, nv)), wrap(fo.narrow(0, 0, nf)), wrap(cid.narrow(0, 0, N))});
}

PyObject* cluster_csr(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor& cid = a.ints("cluster_id");
    const int n_in = rows(cid), n_out = a.i32();
    const at::Tensor off = out_i32({n_out + 1}, cid), mem = out_i32({n_in}, cid);
    checked(c, [&] { return picasso_cluster_csr(c, s, I(cid), n_in, n_out, I(off), I(mem)); });
    return pack({wrap(off), wrap(mem)});
}

PyObject* pool_forward(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const int mode = a.i32();
    const at::Tensor &x = a.f32("x"), &off = a.ints("offsets");
    const at::Tensor *mem = a.maybe_ints("members"), *weight = a.maybe_f32("weight");
    const bool want = a.i32() != 0;
    const int n_in = rows(x), C = rows(x, 1), n_out = rows(off) - 1;
    const at::Tensor y = out_f32({n_out, C}, x), arg = want ? out_i32({n_out, C}, x) : at::Tensor();
    checked(c, [&] { return picasso_pool_forward(c, s, mode, F(x), n_in, C, I(off), I(mem), n_out, F(weight), F(y), want ? I(arg) : nullptr); });
    return want ? pack({wrap(y), wrap(arg)}) : wrap(y);
}

PyObject* pool_backward(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const int mode = a.i32();
    const at::Tensor &gy = a.f32("gy"), &cid = a.ints("cluster_id"), &off = a.ints("offsets");
    const at::Tensor *mem = a.maybe_ints("members"), *weight = a.maybe_f32("weight"), *arg = a.maybe_ints("argmax");
    const int n_in = rows(cid), C = rows(gy, 1), n_out = rows(off) - 1;
    const at::Tensor gx = out_f32({n_in, C}, gy);
    checked(c, [&] { return picasso_pool_backward(c, s, mode, F(gy), n_in, C, I(cid), I(off), I(mem), n_out, F(weight), I(arg), F(gx)); });
    return wrap(gx);
}

PyObject* unpool_forward(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor &y = a.f32("y"), &cid = a.ints("cluster_id");
    const int n_in = rows(cid), C = rows(y, 1);
    const at::Tensor x = out_f32({n_in, C}, y);
    checked(c, [&] { return picasso_unpool_forward(c, s, F(y), n_in, C, I(cid), F(x)); });
    return wrap(x);
}

PyObject* unpool_backward(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor &gx = a.f32("gx"), &off = a.ints("offsets");
    const at::Tensor* mem = a.maybe_ints("members");
    const int n_in = rows(gx), C = rows(gx, 1), n_out = rows(off) - 1;
    const at::Tensor gy = out_f32({n_out, C}, gx);
    checked(c, [&] { return picasso_unpool_backward(c, s, F(gx), n_in, C, I(off), I(mem), n_out, F(gy)); });
    return wrap(gy);
}

PyObject* vertex_corner_csr(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor& f = a.ints("facets");
    const int nF = rows(f), N = a.i32();
    const at::Tensor off = out_i32({N + 1}, f), cor = out_i32({3 * (int64_t)nF}, f);
    checked(c, [&] { return picasso_vertex_corner_csr(c, s, I(f), nF, N, I(off), I(cor)); });
    return pack({wrap(off), wrap(cor)});
}

PyObject* facet_geometry(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor &v = a.f32("verts"), &f = a.ints("facets");
    PyObject* per_mesh = a.next();
    const int alpha = a.i32(), beta = a.i32(), N = rows(v), nF = rows(f);
    std::vector<int32_t> nf;
    if (per_mesh != Py_None) {
        PyObject* seq = PySequence_Fast(per_mesh, "nf: expected a sequence of integers");
        if (!seq) throw PyError{};
        Args items{PySequence_Fast_ITEMS(seq), PySequence_Fast_GET_SIZE(seq)};
        try {
            while (items.at < items.n) nf.push_back(items.i32());
        } catch (const PyError&) {
            Py_DECREF(seq);
            throw;
        }
        Py_DECREF(seq);
    }
    const at::Tensor nrm = out_f32({nF, 3}, v), area = out_f32({nF}, v), lev = out_i32({nF}, v);
    checked(c, [&] {
        return picasso_facet_geometry(c, s, F(v), N, I(f), nF, per_mesh == Py_None ? 1 : (int)nf.size(),
                                      per_mesh == Py_None ? nullptr : nf.data(), alpha, beta, F(nrm), F(area), I(lev));
    });
    return pack({wrap(nrm), wrap(area), wrap(lev)});
}

PyObject* fuzzy_coefficients(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor &nrm = a.f32("normals"), &mu = a.f32("mu");
    const at::Tensor* iv = a.maybe_f32("inv_var");
    const int nF = rows(nrm), T = rows(mu);
    const at::Tensor pi = out_f32({nF, T}, nrm);
    checked(c, [&] { return picasso_fuzzy_coefficients(c, s, F(nrm), nF, F(mu), F(iv), T, F(pi)); });
    return wrap(pi);
}

PyObject* v2f_forward(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor &x = a.f32("x"), &f = a.ints("facets");
    const at::Tensor *level = a.maybe_ints("level"), *w = a.maybe_f32("w"), *out = a.maybe_f32("y");
    const int N = rows(x), C = rows(x, 1), nF = rows(f);
    const at::Tensor y = out ? *out : out_f32({nF, C}, x);
    checked(c, [&] { return picasso_v2f_forward(c, s, F(x), N, C, I(f), nF, I(level), F(w), F(y)); });
    return wrap(y);
}

PyObject* v2f_backward(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor* gy = a.maybe_f32("gy");
    const at::Tensor &x = a.f32("x"), &f = a.ints("facets");
    const at::Tensor *level = a.maybe_ints("level"), *w = a.maybe_f32("w"), *off = a.maybe_ints("offsets"),
                     *cor = a.maybe_ints("corners");
    const int N = rows(x), C = rows(x, 1), nF = rows(f);
    const at::Tensor gx = out_f32({N, C}, x), gw = out_f32({3, C}, x);
    checked(c, [&] { return picasso_v2f_backward(c, s, F(gy), F(x), N, C, I(f), nF, I(level), F(w), I(off), I(cor), F(gx), F(gw)); });
    return pack({wrap(gx), wrap(gw)});
}

PyObject* f2f_forward(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor& tex = a.f32("tex");
    const at::Tensor* bary = a.maybe_f32("bary");
    const at::Tensor& poff = a.ints("poff");
    const at::Tensor* w = a.maybe_f32("w");
    const int P = rows(tex), C = rows(tex, 1), nF = rows(poff) - 1;
    const at::Tensor y = out_f32({nF, C}, tex);
    checked(c, [&] { return picasso_f2f_forward(c, s, F(tex), F(bary), I(poff), nF, P, C, F(w), F(y)); });
    return wrap(y);
}

PyObject* f2f_backward(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor* gy = a.maybe_f32("gy");
    const at::Tensor& tex = a.f32("tex");
    const at::Tensor* bary = a.maybe_f32("bary");
    const at::Tensor& poff = a.ints("poff");
    const at::Tensor* w = a.maybe_f32("w");
    const int P = rows(tex), C = rows(tex, 1), nF = rows(poff) - 1;
    const at::Tensor gtex = out_f32({P, C}, tex), gw = out_f32({3, C}, tex);
    // (rows of points that belong to no facet are zero; only they are written twice)
    checked(c, [&] {
        const int st = picasso_f2f_clear_unowned(c, s, I(poff), nF, P, C, F(gtex));
        return st != PICASSO_OK ? st : picasso_f2f_backward(c, s, F(gy), F(tex), F(bary), I(poff), nF, P, C, F(w), F(gtex), F(gw));
    });
    return pack({wrap(gtex), wrap(gw)});
}

PyObject* f2v_forward(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor &y = a.f32("y"), &pi = a.f32("pi");
    const at::Tensor *w = a.maybe_f32("w"), *off = a.maybe_ints("offsets"), *cor = a.maybe_ints("corners");
    const int N = a.i32();
    const at::Tensor* out = a.maybe_f32("x");
    const int nF = rows(y), C = rows(y, 1), T = rows(pi, 1);
    const at::Tensor x = out ? *out : out_f32({N, C}, y);
    checked(c, [&] { return picasso_f2v_forward(c, s, F(y), nF, C, F(pi), T, F(w), I(off), I(cor), N, F(x)); });
    return wrap(x);
}

PyObject* f2v_backward(Args& a) {
    picasso_ctx* c = a.context();
    void* s = a.stream();
    const at::Tensor &gx = a.f32("gx"), &y = a.f32("y"), &pi = a.f32("pi");
    const at::Tensor *w = a.maybe_f32("w"), *f = a.maybe_ints("facets"), *off = a.maybe_ints("offsets");
    const bool want = a.i32() != 0;
    const int nF = rows(y), C = rows(y, 1), T = rows(pi, 1), N = rows(gx);
    const at::Tensor gy = out_f32({nF, C}, y), gw = out_f32({T, C}, y), gpi = want ? out_f32({nF, T}, y) : at::Tensor();
    checked(c, [&] {
        return picasso_f2v_backward(c, s, F(gx), F(y), nF, C, F(pi), T, F(w), I(f), I(off), N, F(gy), F(gw), want ? F(gpi) : nullptr);
    });
    return pack({wrap(gy), wrap(gw), want ? wrap(gpi) : none()});
}

// (current_device, current_stream, raise): the callables above
PyObject* set_callbacks(Args& a) {
    for (PyObject** p : {&g_current_device, &g_current_stream, &g_raise}) {
        PyObject* o = a.next();
        Py_INCREF(o);
        Py_XDECREF(*p);
        *p = o;
    }
    return none();
}

#define PICASSO_ENTRY(name) {#name, (PyCFunction)(void (*)(void))(PyObject * (*)(PyObject*, PyObject* const*, Py_ssize_t)) & entry<name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    PICASSO_ENTRY(decimate), PICASSO_ENTRY(decimate_batch), PICASSO_ENTRY(cluster_csr), PICASSO_ENTRY(pool_forward),
    PICASSO_ENTRY(pool_backward), PICASSO_ENTRY(unpool_forward), PICASSO_ENTRY(unpool_backward),
    PICASSO_ENTRY(vertex_corner_csr), PICASSO_ENTRY(facet_geometry), PICASSO_ENTRY(fuzzy_coefficients),
    PICASSO_ENTRY(v2f_forward), PICASSO_ENTRY(v2f_backward), PICASSO_ENTRY(f2f_forward), PICASSO_ENTRY(f2f_backward),
    PICASSO_ENTRY(f2v_forward), PICASSO_ENTRY(f2v_backward), PICASSO_ENTRY(set_callbacks), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", "calls of include/picasso.h on torch tensors", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host() { return PyModule_Create(&module); }
