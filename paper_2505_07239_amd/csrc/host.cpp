// Argument checks and marshalling of the calls a layer makes over and over, in native code (the module
// paper_2505_07239_amd._host).
//
// A small layer is bound by the host: seventeen calls of five to eleven microseconds each, of which a launch takes
// 2.8.  The checks of binding.py on tensor attributes, one Python call each, and ctypes took the rest; here a call costs 0.4 to
// 0.9 besides its launches (a gather 5.8 -> 3.5 us, a share product of one launch 8.0 -> 3.2; a layer of seventeen calls
// 139 -> 75 us of host time).
//
// Every function either makes the call or declines by returning None, in which case binding.py takes its own way
// through the same checks and raises what it always raised.  It declines whatever is not plain: other types
// than torch.Tensor itself (subclasses, proxies), tensors without storage or under a functional
// transform, integers that are no int, anything a check of binding.py would refuse.  A return value that is an int is
// the error code of the library.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>

#include "comet_ring.h"

namespace {

// the library's entry points, as the binding loaded them (bind())
struct Library {
    decltype(&comet_set_stream) set_stream;
    decltype(&comet_workspace_bytes) workspace_bytes;
    decltype(&comet_weight_planes_bytes) weight_planes_bytes;
    decltype(&comet_mask_share) mask_share;
    decltype(&comet_open) open;
    decltype(&comet_mask_share_gather) mask_share_gather;
    decltype(&comet_open_weight_planes) open_weight_planes;
    decltype(&comet_open_weight_planes_neuron_major) open_weight_planes_neuron_major;
    decltype(&comet_compact_mask) compact_mask;
    decltype(&comet_somm_share) somm_share;
    decltype(&comet_simm_share) simm_share;
    decltype(&comet_somm_share_unopened) somm_share_unopened;
    decltype(&comet_simm_share_unopened) simm_share_unopened;
    decltype(&comet_share_group) share_group;
} lib;
bool bound = false;
PyTypeObject* planes_type = nullptr;      // binding.WeightPlanes
PyObject *name_buf, *name_shape;

struct Host {
    PyObject_HEAD
    comet_ctx* ctx;
    int device;
};

using at::Tensor;

const Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const Tensor& t = THPVariable_Unpack(o);
    static const c10::DispatchKeySet wrapped = c10::DispatchKeySet(
        {c10::DispatchKey::Python, c10::DispatchKey::Functionalize, c10::DispatchKey::FuncTorchBatched,
         c10::DispatchKey::FuncTorchGradWrapper});
    if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || !t.has_storage() || t.key_set().has_any(wrapped))
        return nullptr;
    return &t;
}
const Tensor* typed(PyObject* o, c10::ScalarType type) {
    const Tensor* t = plain(o);
    return t && t->scalar_type() == type && t->is_contiguous() ? t : nullptr;
}
const Tensor* words(PyObject* o) { return typed(o, c10::kLong); }

bool integer(PyObject* o, long long lo, long long hi, long long* v) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &over);
    return !over && *v >= lo && *v <= hi;
}
bool flag(PyObject* o, bool* v) {
    *v = o == Py_True;
    return *v || o == Py_False;
}
bool shaped(const Tensor& t, int64_t r, int64_t c) { return t.dim() == 2 && t.size(0) == r && t.size(1) == c; }

constexpr long long INT_LIMIT = 0x7fffffff;
uint64_t* u64(const Tensor& t) { return static_cast<uint64_t*>(t.data_ptr()); }

// what the calls over an index list have in common
struct Index {
    long long bs, cap;
    const int32_t* idx;
    const int32_t* n;
    bool read(PyObject* o_bs, PyObject* o_idx, PyObject* o_n, PyObject* o_cap, bool required) {
        if (!integer(o_bs, 1, INT_LIMIT, &bs) || !integer(o_cap, 0, INT_LIMIT, &cap)) return false;
        idx = n = nullptr;
        if (o_n != Py_None) {
            const Tensor* t = plain(o_n);
            if (!t || t->scalar_type() != c10::kInt || t->numel() < 1) return false;
            n = static_cast<const int32_t*>(t->data_ptr());
        }
        if (o_idx == Py_None) return !required;
        const Tensor* t = typed(o_idx, c10::kInt);
        if (!t || (!n && t->numel() < cap)) return false;
        idx = static_cast<const int32_t*>(t->data_ptr());
        return true;
    }
    int64_t ld() const { return bs * cap; }
};

// a weight-side operand: words, or planes (a raw buffer and the shape it stands for)
struct Weights {
    int64_t rows, cols;
    const uint64_t* data;
    bool planes;
    bool read(PyObject* o) {
        planes = Py_TYPE(o) == planes_type;
        if (!planes) {
            const Tensor* t = words(o);
            if (!t || t->dim() != 2) return false;
            rows = t->size(0); cols = t->size(1); data = u64(*t);
            return true;
        }
        THPObjectPtr buf(PyObject_GetAttr(o, name_buf)), shape(PyObject_GetAttr(o, name_shape));
        bool ok = buf && shape && PyTuple_CheckExact(shape.get()) && PyTuple_GET_SIZE(shape.get()) == 2;
        long long r = 0, c = 0;
        ok = ok && integer(PyTuple_GET_ITEM(shape.get(), 0), 0, 1ll << 40, &r) &&
             integer(PyTuple_GET_ITEM(shape.get(), 1), 0, 1ll << 40, &c);
        const Tensor* t = ok ? plain(buf) : nullptr;
        if (t) data = u64(*t);             // (the planes object holds the buffer)
        rows = r; cols = c;
        PyErr_Clear();
        return t != nullptr;
    }
    bool is(int64_t r, int64_t c) const { return rows == r && cols == c; }
};

// The result: the caller's tensor of this shape, or a new one; null to decline.  (References that a call owns are
// THPObjectPtr throughout: an allocation or a stream lookup that throws gives them back.)
THPObjectPtr result(PyObject* o, int64_t rows, int64_t cols, const Tensor& like, uint64_t** data) {
    if (o == Py_None) {
        Tensor t = at::empty({rows, cols}, like.options().requires_grad(false));
        *data = u64(t);
        return THPObjectPtr(THPVariable_Wrap(std::move(t)));
    }
    const Tensor* t = words(o);
    if (!t || !shaped(*t, rows, cols)) return THPObjectPtr();
    *data = u64(*t);
    return THPObjectPtr::dup(o);
}

// a workspace of at least `need` bytes: the context's, or decline
bool scratch(PyObject* o, size_t need, void** ws) {
    *ws = nullptr;
    if (need == 0) return true;
    const Tensor* t = plain(o);
    if (!t || t->scalar_type() != c10::kByte || (size_t)t->numel() < need) return false;
    *ws = t->data_ptr();
    return true;
}

// On torch's current stream, without the interpreter lock (as ctypes calls).  `out` is what the call returns.
template <class F>
PyObject* call(Host* self, THPObjectPtr out, F&& f) {
    void* stream = c10::hip::getCurrentHIPStream((c10::DeviceIndex)self->device).stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = lib.set_stream(self->ctx, stream);
    if (rc == 0) rc = f();
    Py_END_ALLOW_THREADS
    return rc == 0 ? out.release() : PyLong_FromLong(rc);
}

#define DECLINE Py_RETURN_NONE
#define READY(nargs_wanted) if (!bound || !self->ctx || nargs != (nargs_wanted)) DECLINE

// (open?, a, b, out)
PyObject* elementwise(Host* self, PyObject* const* arg, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    READY(4);
    bool open;
    const Tensor *a = words(arg[1]), *b = words(arg[2]);
    if (!flag(arg[0], &open) || !a || !b || a->numel() != b->numel()) DECLINE;
    THPObjectPtr out;
    uint64_t* o;
    if (arg[3] == Py_None) {
        Tensor t = at::empty(a->sizes(), a->options().requires_grad(false));
        o = u64(t);
        out = THPVariable_Wrap(std::move(t));
    } else {
        const Tensor* t = words(arg[3]);
        if (!t || t->numel() != a->numel()) DECLINE;
        o = u64(*t);
        out = THPObjectPtr::dup(arg[3]);
    }
    const uint64_t *pa = u64(*a), *pb = u64(*b);
    const size_t n = (size_t)a->numel();
    return call(self, std::move(out), [&] { return open ? lib.open(self->ctx, pa, pb, o, n) : lib.mask_share(self->ctx, pa, pb, o, n); });
    END_HANDLE_TH_ERRORS
}

// (w, b, axis, bs, idx, n, cap, out)
PyObject* gather(Host* self, PyObject* const* arg, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    READY(8);
    const Tensor *w = words(arg[0]), *b = words(arg[1]);
    long long axis;
    Index ix;
    if (!w || !b || w->dim() != 2 || !integer(arg[2], 0, 1, &axis) || !ix.read(arg[3], arg[4], arg[5], arg[6], true) ||
        !shaped(*b, w->size(0), w->size(1)))
        DECLINE;
    const int64_t rows = w->size(0), cols = w->size(1);
    uint64_t* o;
    THPObjectPtr out = axis == COMET_AXIS_COLS ? result(arg[7], rows, ix.ld(), *w, &o) : result(arg[7], ix.ld(), cols, *w, &o);
    if (!out) DECLINE;
    const uint64_t *pw = u64(*w), *pb = u64(*b);
    return call(self, std::move(out), [&] {
        return lib.mask_share_gather(self->ctx, pw, pb, o, rows, cols, (int)axis, (int)ix.bs, ix.idx, ix.n, (int)ix.cap);
    });
    END_HANDLE_TH_ERRORS
}

// (g_0, g_1, out, neuron_major) -> the buffer of planes
PyObject* open_planes(Host* self, PyObject* const* arg, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    READY(4);
    bool nm;
    const Tensor* g0 = words(arg[0]);
    const Tensor* g1 = arg[1] == Py_None ? nullptr : words(arg[1]);
    if (!g0 || g0->dim() != 2 || !flag(arg[3], &nm) || (arg[1] != Py_None && (!g1 || !g1->sizes().equals(g0->sizes())))) DECLINE;
    const int64_t k = g0->size(nm ? 1 : 0), n = g0->size(nm ? 0 : 1);
    const size_t need = lib.weight_planes_bytes(k, n);
    THPObjectPtr out;
    void* o;
    if (arg[2] == Py_None) {
        Tensor t = at::empty({(int64_t)(need < 16 ? 16 : need)}, g0->options().dtype(c10::kByte).requires_grad(false));
        o = t.data_ptr();
        out = THPVariable_Wrap(std::move(t));
    } else {
        const Tensor* t = plain(arg[2]);
        if (!t || t->scalar_type() != c10::kByte || (size_t)t->numel() < need) DECLINE;
        o = t->data_ptr();
        out = THPObjectPtr::dup(arg[2]);
    }
    const uint64_t *p0 = u64(*g0), *p1 = g1 ? u64(*g1) : nullptr;
    return call(self, std::move(out), [&] {
        return nm ? lib.open_weight_planes_neuron_major(self->ctx, p0, p1, k, n, o) : lib.open_weight_planes(self->ctx, p0, p1, k, n, o);
    });
    END_HANDLE_TH_ERRORS
}

// (ws, mask, idx, n) -> True
PyObject* compact(Host* self, PyObject* const* arg, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    READY(4);
    const Tensor *mask = typed(arg[1], c10::kByte), *idx = plain(arg[2]), *n = plain(arg[3]);
    if (!mask || !idx || !n || mask->dim() < 1 || mask->dim() > 2) DECLINE;
    const int64_t n_tok = mask->dim() == 2 ? mask->size(0) : 1, nb = mask->size(mask->dim() - 1);
    const size_t need = lib.workspace_bytes(COMET_OP_COMPACT, n_tok, 0, nb, 0);
    void* ws;
    if (!scratch(arg[0], need, &ws)) DECLINE;
    auto* m = static_cast<const uint8_t*>(mask->data_ptr());
    auto *pi = static_cast<int32_t*>(idx->data_ptr()), *pn = static_cast<int32_t*>(n->data_ptr());
    return call(self, THPObjectPtr::dup(Py_True), [&] { return lib.compact_mask(self->ctx, m, n_tok, nb, pi, pn, ws, need); });
    END_HANDLE_TH_ERRORS
}

// One share product: operands, shapes and flags (binding.py: _somm_shapes, _simm_shapes).
struct Product {
    bool somm;
    int64_t m, k, n, zr, zc;       // k, n as the library's call takes them; the result's shape
    int flags;
    const uint64_t *e, *f, *a, *b, *c;
    const Tensor* like;
    bool read(bool somm_, const Index& ix, PyObject* oe, PyObject* of, PyObject* oa, PyObject* ob, PyObject* oc, bool a_full,
              bool b_full, bool nm) {
        somm = somm_;
        const Tensor *te = words(oe), *ta = words(oa), *tc = words(oc);
        Weights wf, wb;
        if (!te || !ta || !tc || te->dim() != 2 || ta->dim() != 2 || !wf.read(of) || !wb.read(ob) || wf.planes != wb.planes)
            return false;
        const int64_t ld = ix.ld();
        auto as = [&](const Weights& w, int64_t r, int64_t c) { return nm ? w.is(c, r) : w.is(r, c); };
        m = te->size(0);
        if (somm) {
            k = te->size(1);
            n = b_full ? (nm ? wb.rows : wb.cols) : 0;
            zr = m; zc = ld;
            if (!as(wf, k, ld) || !shaped(*ta, m, k) || !as(wb, k, b_full ? n : ld)) return false;
            flags = (b_full ? COMET_FULL_B : 0) | (nm ? COMET_WEIGHTS_NEURON_MAJOR : 0);
        } else {
            n = wf.cols;
            k = a_full ? ta->size(1) : b_full ? wb.rows : 0;
            zr = m; zc = n;
            if (!shaped(*te, m, ld) || !wf.is(ld, n) || !shaped(*ta, m, a_full ? k : ld) || !wb.is(b_full ? k : ld, n)) return false;
            flags = (a_full ? COMET_FULL_A : 0) | (b_full ? COMET_FULL_B : 0);
        }
        if (!shaped(*tc, zr, zc)) return false;
        if (wf.planes) flags |= COMET_WEIGHT_PLANES;
        e = u64(*te); f = wf.data; a = u64(*ta); b = wb.data; c = u64(*tc);
        like = te;
        return true;
    }
    size_t workspace(const Index& ix) const {
        return somm ? lib.workspace_bytes(COMET_OP_SOMM, m, k, ix.ld(), (int)ix.bs)
                    : lib.workspace_bytes(COMET_OP_SIMM, m, ix.ld(), n, (int)ix.bs);
    }
};

// (ws, somm?, party, bs, idx, n, cap, e, f, g_1 or None, a, b, c, a_full, b_full, neuron_major, out): with g_1 the unopened form
PyObject* share(Host* self, PyObject* const* arg, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    READY(17);
    bool somm, a_full, b_full, nm;
    long long party;
    Index ix;
    Product p;
    if (!flag(arg[1], &somm) || !integer(arg[2], 0, 1, &party) || !flag(arg[13], &a_full) || !flag(arg[14], &b_full) ||
        !flag(arg[15], &nm) || !ix.read(arg[3], arg[4], arg[5], arg[6], b_full || (!somm && a_full)) ||
        !p.read(somm, ix, arg[7], arg[8], arg[10], arg[11], arg[12], a_full, b_full, nm))
        DECLINE;
    const uint64_t* g1 = nullptr;
    if (arg[9] != Py_None) {
        Weights w;
        if ((p.flags & COMET_WEIGHT_PLANES) || nm || !w.read(arg[9]) || w.planes || !(somm ? w.is(p.k, ix.ld()) : w.is(ix.ld(), p.n))) DECLINE;
        g1 = w.data;
    }
    const size_t need = p.workspace(ix);
    void* ws;
    if (!scratch(arg[0], need, &ws)) DECLINE;
    uint64_t* z;
    THPObjectPtr out = result(arg[16], p.zr, p.zc, *p.like, &z);
    if (!out) DECLINE;
    return call(self, std::move(out), [&] {
        const int bs = (int)ix.bs, cap = (int)ix.cap;
        if (g1 && somm)
            return lib.somm_share_unopened(self->ctx, (int)party, p.m, p.k, p.n, bs, ix.idx, ix.n, cap, p.flags, p.e, p.f, g1, p.a, p.b, p.c, z, ws, need);
        if (g1)
            return lib.simm_share_unopened(self->ctx, (int)party, p.m, p.k, p.n, bs, ix.idx, ix.n, cap, p.flags, p.e, p.f, g1, p.a, p.b, p.c, z, ws, need);
        if (somm)
            return lib.somm_share(self->ctx, (int)party, p.m, p.k, p.n, bs, ix.idx, ix.n, cap, p.flags, p.e, p.f, p.a, p.b, p.c, z, ws, need);
        return lib.simm_share(self->ctx, (int)party, p.m, p.k, p.n, bs, ix.idx, ix.n, cap, p.flags, p.e, p.f, p.a, p.b, p.c, z, ws, need);
    });
    END_HANDLE_TH_ERRORS
}

// (ws, somm?, bs, idx, n, cap, members, a_full, b_full, out or None) -> list of results
PyObject* group(Host* self, PyObject* const* arg, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    READY(10);
    bool somm, a_full, b_full;
    Index ix;
    PyObject *members = arg[6], *given = arg[9];
    if (!flag(arg[1], &somm) || !flag(arg[7], &a_full) || !flag(arg[8], &b_full) ||
        !ix.read(arg[2], arg[3], arg[4], arg[5], b_full || (!somm && a_full)) || !PyList_CheckExact(members) ||
        (given != Py_None && !PyList_CheckExact(given)))
        DECLINE;
    const Py_ssize_t count = PyList_GET_SIZE(members);
    if (count < 1 || count > COMET_SHARE_GROUP_MAX || (given != Py_None && PyList_GET_SIZE(given) < count)) DECLINE;
    Product p0 = {};
    comet_share_operands ops[COMET_SHARE_GROUP_MAX] = {};
    long long party;
    for (Py_ssize_t j = 0; j < count; ++j) {
        PyObject* t = PyList_GET_ITEM(members, j);
        Product p;
        if (!PyTuple_CheckExact(t) || PyTuple_GET_SIZE(t) != 6 || !integer(PyTuple_GET_ITEM(t, 0), 0, 1, &party) ||
            !p.read(somm, ix, PyTuple_GET_ITEM(t, 1), PyTuple_GET_ITEM(t, 2), PyTuple_GET_ITEM(t, 3), PyTuple_GET_ITEM(t, 4),
                    PyTuple_GET_ITEM(t, 5), a_full, b_full, false))
            DECLINE;
        if (j == 0) p0 = p;
        else if (p.m != p0.m || p.k != p0.k || p.n != p0.n || p.flags != p0.flags) DECLINE;
        ops[j] = {(int32_t)party, 0, p.e, p.f, p.a, p.b, p.c, nullptr};
    }
    const size_t need = p0.workspace(ix) * (size_t)count;
    void* ws;
    if (!scratch(arg[0], need, &ws)) DECLINE;
    THPObjectPtr outs(PyList_New(count));
    if (!outs) return nullptr;
    for (Py_ssize_t j = 0; j < count; ++j) {
        if (given != Py_None && PyList_GET_ITEM(given, j) == Py_None) DECLINE;   // (no result of its own for one member of a list)
        THPObjectPtr z = result(given == Py_None ? Py_None : PyList_GET_ITEM(given, j), p0.zr, p0.zc, *p0.like, &ops[j].Z_i);
        if (!z) DECLINE;
        PyList_SET_ITEM(outs.get(), j, z.release());
    }
    return call(self, std::move(outs), [&] {
        return lib.share_group(self->ctx, somm ? COMET_OP_SOMM : COMET_OP_SIMM, (int)count, ops, p0.m, p0.k, p0.n, (int)ix.bs, ix.idx,
                               ix.n, (int)ix.cap, p0.flags, ws, need);
    });
    END_HANDLE_TH_ERRORS
}

// ---------------------------------------------------------------------------
// the type and the module
// ---------------------------------------------------------------------------
PyObject* host_new(PyTypeObject* type, PyObject* args, PyObject*) {
    unsigned long long ctx;
    int device;
    if (!PyArg_ParseTuple(args, "Ki", &ctx, &device)) return nullptr;
    Host* self = reinterpret_cast<Host*>(type->tp_alloc(type, 0));
    if (!self) return nullptr;
    self->ctx = reinterpret_cast<comet_ctx*>(ctx);
    self->device = device;
    return reinterpret_cast<PyObject*>(self);
}

PyObject* host_close(Host* self, PyObject*) {
    self->ctx = nullptr;
    Py_RETURN_NONE;
}

template <PyObject* (*F)(Host*, PyObject* const*, Py_ssize_t)>
PyObject* entry(PyObject* self, PyObject* const* arg, Py_ssize_t nargs) { return F(reinterpret_cast<Host*>(self), arg, nargs); }
#define ENTRY(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<f>)), METH_FASTCALL, nullptr}

PyMethodDef host_methods[] = {ENTRY(elementwise), ENTRY(gather), ENTRY(open_planes), ENTRY(compact), ENTRY(share), ENTRY(group),
                              {"close", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&host_close)), METH_NOARGS, nullptr},
                              {nullptr, nullptr, 0, nullptr}};

PyTypeObject host_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// bind(addresses of the entry points by name, the class of weight planes)
PyObject* bind(PyObject*, PyObject* args) {
    PyObject *table, *planes;
    if (!PyArg_ParseTuple(args, "O!O!", &PyDict_Type, &table, &PyType_Type, &planes)) return nullptr;
    auto find = [&](const char* name, auto& f) {
        PyObject* v = PyDict_GetItemString(table, name);
        void* a = v ? PyLong_AsVoidPtr(v) : nullptr;
        if (!a) {
            if (!PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "no address for %s", name);
            return false;
        }
        f = reinterpret_cast<std::remove_reference_t<decltype(f)>>(a);
        return true;
    };
    bound = find("comet_set_stream", lib.set_stream) && find("comet_workspace_bytes", lib.workspace_bytes) &&
            find("comet_weight_planes_bytes", lib.weight_planes_bytes) && find("comet_mask_share", lib.mask_share) &&
            find("comet_open", lib.open) && find("comet_mask_share_gather", lib.mask_share_gather) &&
            find("comet_open_weight_planes", lib.open_weight_planes) &&
            find("comet_open_weight_planes_neuron_major", lib.open_weight_planes_neuron_major) &&
            find("comet_compact_mask", lib.compact_mask) && find("comet_somm_share", lib.somm_share) &&
            find("comet_simm_share", lib.simm_share) && find("comet_somm_share_unopened", lib.somm_share_unopened) &&
            find("comet_simm_share_unopened", lib.simm_share_unopened) && find("comet_share_group", lib.share_group);
    if (!bound) return nullptr;
    Py_INCREF(planes);
    Py_XDECREF(planes_type);
    planes_type = reinterpret_cast<PyTypeObject*>(planes);
    Py_RETURN_NONE;
}

PyMethodDef module_methods[] = {{"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, module_methods};

}  // namespace

PyMODINIT_FUNC PyInit__host() {
    host_type.tp_name = "paper_2505_07239_amd._host.Host";
    host_type.tp_basicsize = sizeof(Host);
    host_type.tp_flags = Py_TPFLAGS_DEFAULT;
    host_type.tp_methods = host_methods;
    host_type.tp_new = host_new;
    if (PyType_Ready(&host_type) < 0) return nullptr;
    name_buf = PyUnicode_InternFromString("buf");
    name_shape = PyUnicode_InternFromString("shape");
    PyObject* m = PyModule_Create(&module_def);
    if (!m || !name_buf || !name_shape) return nullptr;
    Py_INCREF(&host_type);
    if (PyModule_AddObject(m, "Host", reinterpret_cast<PyObject*>(&host_type)) < 0) return nullptr;
    return m;
}
