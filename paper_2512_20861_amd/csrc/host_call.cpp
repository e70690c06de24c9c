// The launching functions of the Python binding as native callables.
//
// What bounds a call of few tokens is the host: a marshaller in Python (shape, type and device checks, pointers, the
// current stream, a foreign-function call) takes 11 us where the GPU needs 9 for both kernels of a 4096 x 4096 Monarch
// layer. A Launcher does the same checks on the tensors' own C++ objects and calls the C ABI directly, about 1 us.
// It only serves calls whose arguments are exactly right; anything else (a shape that does not fit, another type, a
// missing workspace, an explicit stream object) goes to the Python marshaller, which is the one place that says what
// is wrong and allocates what is missing. Arguments, defaults, results and errors are therefore those of the
// marshaller in every case.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>

#include <cstring>
#include <string>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/blr.h"

namespace {

constexpr int kMaxParams = 11;
constexpr int kNotServed = -1;          // the Python marshaller takes the call

// the call itself runs without the interpreter lock, as a foreign-function call does
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// the arguments of one call, by position in the parameter list (nullptr: not given)
struct Args { PyObject* v[kMaxParams]; };

// one tensor argument; ok() is false for anything but a contiguous GPU tensor
struct Tensor {
    const at::Tensor* t = nullptr;
    explicit Tensor(PyObject* o) {
        if (o && THPVariable_Check(o)) {
            const at::Tensor& x = THPVariable_Unpack(o);
            if (x.is_cuda() && x.is_contiguous()) t = &x;
        }
    }
    bool ok() const { return t != nullptr; }
    bool like(const Tensor& o) const { return t->scalar_type() == o.t->scalar_type() && t->device() == o.t->device(); }
    bool shape(std::initializer_list<int64_t> want) const { return t->sizes().equals(at::IntArrayRef(want)); }
    int64_t dim(int i) const { return t->size(i); }
    bool dims(int n) const { return t->dim() == n; }
    bool bytes_on(const Tensor& o) const { return t->scalar_type() == at::kByte && t->device() == o.t->device(); }
    void* ptr() const { return t->data_ptr(); }
    int64_t numel() const { return t->numel(); }
};

bool dtype_of(const Tensor& x, blr_dtype* dt) {
    if (x.t->scalar_type() == at::kBFloat16) { *dt = BLR_BF16; return true; }
    if (x.t->scalar_type() == at::kFloat) { *dt = BLR_F32; return true; }
    return false;
}

bool whole(PyObject* o, long lo, long hi, long* out) {
    if (!o || !PyLong_CheckExact(o)) return false;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v < lo || v > hi) return false;
    *out = v;
    return true;
}
bool positive(PyObject* o, int* out) {
    long v;
    if (!whole(o, 1, 0x7fffffff, &v)) return false;
    *out = (int)v;
    return true;
}
bool flag_bits(PyObject* o, unsigned* out) {
    long v = 0;
    if (o && !whole(o, 0, 0xffffffffL, &v)) return false;
    *out = (unsigned)v;
    return true;
}
// the stream argument: not given (or None) is the stream that is current now
bool stream_of(PyObject* o, blr_stream* out) {
    if (o && o != Py_None) return false;
    *out = (blr_stream)c10::hip::getCurrentHIPStream().stream();
    return true;
}
bool fits_int(int64_t n) { return n > 0 && n <= 0x7fffffff; }

// X[T][n_in], Y[T][n_out] of one storage type and device
struct InOut {
    Tensor X, Y;
    int64_t T = 0;
    int n_in = 0, n_out = 0;
    blr_dtype dt{};
    bool good = false;
    InOut(PyObject* x, PyObject* y) : X(x), Y(y) {
        if (!X.ok() || !Y.ok() || !X.dims(2) || !Y.dims(2) || !Y.like(X) || !dtype_of(X, &dt)) return;
        T = X.dim(0);
        if (Y.dim(0) != T || !fits_int(X.dim(1)) || !fits_int(Y.dim(1))) return;
        n_in = (int)X.dim(1);
        n_out = (int)Y.dim(1);
        good = true;
    }
};

bool workspace(PyObject* o, const Tensor& X, Tensor* ws) {
    *ws = Tensor(o);
    return ws->ok() && ws->bytes_on(X);
}

// R[b_in][r_block b_out][n_in/b_in], L[b_out][n_out/b_out][b_in r_block]
bool monarch_factors(const InOut& io, const Tensor& R, const Tensor& L, int b_in, int b_out, int64_t r_block) {
    return R.ok() && L.ok() && R.like(io.X) && L.like(io.X) && io.n_in % b_in == 0 && io.n_out % b_out == 0 &&
           R.shape({b_in, r_block * b_out, io.n_in / b_in}) && L.shape({b_out, io.n_out / b_out, b_in * r_block});
}

int monarch_forward(const Args& a) {                     // X, R, L, Y, nblocks, r, flags, workspace, stream
    InOut io(a.v[0], a.v[3]);
    Tensor R(a.v[1]), L(a.v[2]), ws(nullptr);
    int nb, r;
    unsigned flags;
    blr_stream s;
    if (!io.good || !positive(a.v[4], &nb) || !positive(a.v[5], &r) || r % nb || !flag_bits(a.v[6], &flags) || !workspace(a.v[7], io.X, &ws) ||
        !stream_of(a.v[8], &s) || !monarch_factors(io, R, L, nb, nb, r / nb)) return kNotServed;
    Unlocked unlocked;
    return blr_monarch_forward(io.X.ptr(), R.ptr(), L.ptr(), io.Y.ptr(), io.T, io.n_in, io.n_out, nb, r, io.dt, flags, ws.ptr(), (size_t)ws.numel(), s);
}

int monarch_forward_static(const Args& a) {              // X, R, L, Y, nblocks, r, flags, stream
    InOut io(a.v[0], a.v[3]);
    Tensor R(a.v[1]), L(a.v[2]);
    int nb, r;
    unsigned flags;
    blr_stream s;
    if (!io.good || !positive(a.v[4], &nb) || !positive(a.v[5], &r) || r % nb || !flag_bits(a.v[6], &flags) || !stream_of(a.v[7], &s) ||
        !monarch_factors(io, R, L, nb, nb, r / nb)) return kNotServed;
    Unlocked unlocked;
    return blr_monarch_forward_static(io.X.ptr(), R.ptr(), L.ptr(), io.Y.ptr(), io.T, io.n_in, io.n_out, nb, r, io.dt, flags, s);
}

int monarch_rect_forward(const Args& a) {                // X, R, L, Y, b_in, b_out, r_block, flags, workspace, stream
    InOut io(a.v[0], a.v[3]);
    Tensor R(a.v[1]), L(a.v[2]), ws(nullptr);
    int b_in, b_out, rb;
    unsigned flags;
    blr_stream s;
    if (!io.good || !positive(a.v[4], &b_in) || !positive(a.v[5], &b_out) || !positive(a.v[6], &rb) || !flag_bits(a.v[7], &flags) ||
        !workspace(a.v[8], io.X, &ws) || !stream_of(a.v[9], &s) || !monarch_factors(io, R, L, b_in, b_out, rb)) return kNotServed;
    Unlocked unlocked;
    return blr_monarch_rect_forward(io.X.ptr(), R.ptr(), L.ptr(), io.Y.ptr(), io.T, io.n_in, io.n_out, b_in, b_out, rb, io.dt, flags, ws.ptr(), (size_t)ws.numel(), s);
}

int lowrank_forward(const Args& a) {                     // X, V, U, Y, flags, workspace, stream
    InOut io(a.v[0], a.v[3]);
    Tensor V(a.v[1]), U(a.v[2]), ws(nullptr);
    unsigned flags;
    blr_stream s;
    if (!io.good || !V.ok() || !U.ok() || !V.like(io.X) || !U.like(io.X) || !U.dims(2) || !fits_int(U.dim(1)) || !flag_bits(a.v[4], &flags) ||
        !workspace(a.v[5], io.X, &ws) || !stream_of(a.v[6], &s)) return kNotServed;
    const int r = (int)U.dim(1);
    if (U.dim(0) != io.n_out || !V.shape({r, io.n_in})) return kNotServed;
    Unlocked unlocked;
    return blr_lowrank_forward(io.X.ptr(), V.ptr(), U.ptr(), io.Y.ptr(), io.T, io.n_in, io.n_out, r, io.dt, flags, ws.ptr(), (size_t)ws.numel(), s);
}

int blast_forward(const Args& a) {                       // X, U, S, V, Y, b, r, flags, workspace, stream
    InOut io(a.v[0], a.v[4]);
    Tensor U(a.v[1]), V(a.v[3]), ws(nullptr);
    int b, r;
    unsigned flags;
    blr_stream s;
    if (!io.good || !U.ok() || !V.ok() || !U.like(io.X) || !positive(a.v[5], &b) || !positive(a.v[6], &r) || !flag_bits(a.v[7], &flags) ||
        !workspace(a.v[8], io.X, &ws) || !stream_of(a.v[9], &s) || io.n_in % b || io.n_out % b || !U.shape({b, io.n_out / b, r})) return kNotServed;
    const void* S = nullptr;
    if (flags & BLR_BLAST_PACKED) {
        if (a.v[2] != Py_None || !V.bytes_on(io.X)) return kNotServed;
        const size_t need = blr_blast_packed_bytes(io.n_in, io.n_out, b, r, io.dt);
        if ((size_t)V.numel() < (need > 16 ? need : 16)) return kNotServed;
    } else {
        Tensor St(a.v[2]);
        if (!St.ok() || !St.like(io.X) || !V.like(io.X) || !St.shape({b, b, r}) || !V.shape({b, io.n_in / b, r})) return kNotServed;
        S = St.ptr();
    }
    Unlocked unlocked;
    return blr_blast_forward(io.X.ptr(), U.ptr(), S, V.ptr(), io.Y.ptr(), io.T, io.n_in, io.n_out, b, r, io.dt, flags, ws.ptr(), (size_t)ws.numel(), s);
}

int blast_group_forward(const Args& a) {                 // X, U, packed, Y, b, r, members, flags, workspace, stream
    InOut io(a.v[0], a.v[3]);
    Tensor U(a.v[1]), P(a.v[2]), ws(nullptr);
    int b, r, members;
    unsigned flags;
    blr_stream s;
    if (!io.good || !U.ok() || !P.ok() || !U.like(io.X) || !P.bytes_on(io.X) || !positive(a.v[4], &b) || !positive(a.v[5], &r) ||
        !positive(a.v[6], &members) || !flag_bits(a.v[7], &flags) || !workspace(a.v[8], io.X, &ws) || !stream_of(a.v[9], &s)) return kNotServed;
    if (io.n_out % members || (int64_t)r * members > 0x7fffffff) return kNotServed;
    const int n_out = io.n_out / members;
    if (n_out % b || !U.shape({members, b, n_out / b, r})) return kNotServed;
    const size_t need = blr_blast_packed_bytes(io.n_in, n_out, b, members * r, io.dt);
    if ((size_t)P.numel() < (need > 16 ? need : 16)) return kNotServed;
    Unlocked unlocked;
    return blr_blast_group_forward(io.X.ptr(), U.ptr(), P.ptr(), io.Y.ptr(), io.T, io.n_in, n_out, b, r, members, io.dt, flags, ws.ptr(), (size_t)ws.numel(), s);
}

int dense_reference_forward(const Args& a) {             // X, W, Y, flags, stream
    InOut io(a.v[0], a.v[2]);
    Tensor W(a.v[1]);
    unsigned flags;
    blr_stream s;
    if (!io.good || !W.ok() || !W.like(io.X) || !flag_bits(a.v[3], &flags) || !stream_of(a.v[4], &s) || !W.shape({io.n_out, io.n_in})) return kNotServed;
    Unlocked unlocked;
    return blr_dense_reference_forward(io.X.ptr(), W.ptr(), io.Y.ptr(), io.T, io.n_in, io.n_out, io.dt, flags, s);
}

struct Entry {
    const char* name;
    int (*serve)(const Args&);
    int n_params, result;                                // result: which argument the call returns
    const char* params[kMaxParams];
};

const Entry kEntries[] = {
    {"monarch_forward", monarch_forward, 9, 3, {"X", "R", "L", "Y", "nblocks", "r", "flags", "workspace", "stream"}},
    {"monarch_forward_static", monarch_forward_static, 8, 3, {"X", "R", "L", "Y", "nblocks", "r", "flags", "stream"}},
    {"monarch_rect_forward", monarch_rect_forward, 10, 3, {"X", "R", "L", "Y", "b_in", "b_out", "r_block", "flags", "workspace", "stream"}},
    {"lowrank_forward", lowrank_forward, 7, 3, {"X", "V", "U", "Y", "flags", "workspace", "stream"}},
    {"blast_forward", blast_forward, 10, 4, {"X", "U", "S", "V", "Y", "b", "r", "flags", "workspace", "stream"}},
    {"blast_group_forward", blast_group_forward, 10, 3, {"X", "U", "packed", "Y", "b", "r", "members", "flags", "workspace", "stream"}},
    {"dense_reference_forward", dense_reference_forward, 5, 2, {"X", "W", "Y", "flags", "stream"}},
};

// A launching function: served natively where the arguments are exactly right, else by `fallback`
struct Launcher {
    PyObject_HEAD
    PyObject* dict;
    PyObject* fallback;                                  // the call through the Python marshaller
    PyObject* failed;                                    // failed(status, name) raises
    const Entry* entry;
    PyObject* names[kMaxParams];                         // interned parameter names
    PyObject* weakrefs;
    vectorcallfunc vectorcall;
};

PyObject* launcher_call(PyObject* self_, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
    Launcher* self = (Launcher*)self_;
    const Entry& e = *self->entry;
    const Py_ssize_t n = PyVectorcall_NARGS(nargsf), nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    int st = kNotServed;
    Args a{};
    bool plain = n <= e.n_params;
    if (plain) {
        for (Py_ssize_t i = 0; i < n; ++i) a.v[i] = args[i];
        for (Py_ssize_t k = 0; k < nkw && plain; ++k) {
            PyObject* name = PyTuple_GET_ITEM(kwnames, k);
            int at = -1;
            for (int i = 0; i < e.n_params; ++i)         // keywords of a call site are interned: identity nearly always decides
                if (name == self->names[i]) { at = i; break; }
            plain = at >= n && !a.v[at];                 // anything odd (unknown, given twice): the marshaller says so
            if (plain) a.v[at] = args[n + k];
        }
    }
    if (plain) {
        try {
            st = e.serve(a);
        } catch (const std::exception&) {                // no such tensor storage, no device: the marshaller reports it
            st = kNotServed;
        }
    }
    if (st == BLR_OK) {
        PyObject* y = a.v[e.result];
        Py_INCREF(y);
        return y;
    }
    if (st == kNotServed) return PyObject_Vectorcall(self->fallback, args, nargsf, kwnames);
    return PyObject_CallFunction(self->failed, "is", st, (std::string("blr_") + e.name).c_str());
}

void launcher_dealloc(PyObject* self_) {
    Launcher* self = (Launcher*)self_;
    PyObject_GC_UnTrack(self_);
    if (self->weakrefs) PyObject_ClearWeakRefs(self_);
    Py_XDECREF(self->dict);
    Py_XDECREF(self->fallback);
    Py_XDECREF(self->failed);
    for (PyObject* n : self->names) Py_XDECREF(n);
    PyObject_GC_Del(self_);
}
int launcher_traverse(PyObject* self_, visitproc visit, void* arg) {
    Launcher* self = (Launcher*)self_;
    Py_VISIT(self->dict);
    Py_VISIT(self->fallback);
    Py_VISIT(self->failed);
    return 0;
}

PyTypeObject LauncherType = {PyVarObject_HEAD_INIT(nullptr, 0)};

// a copy of a function is the function
PyObject* launcher_itself(PyObject* self, PyObject*) {
    Py_INCREF(self);
    return self;
}
PyMethodDef launcher_methods[] = {{"__copy__", launcher_itself, METH_NOARGS, nullptr}, {"__deepcopy__", launcher_itself, METH_O, nullptr}, {}};
PyGetSetDef launcher_getset[] = {{"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, nullptr, nullptr}, {}};

// launcher(name, fallback, failed) -> Launcher, or None for a function without a native form
PyObject* make_launcher(PyObject*, PyObject* args) {
    const char* name;
    PyObject *fallback, *failed;
    if (!PyArg_ParseTuple(args, "sOO", &name, &fallback, &failed)) return nullptr;
    for (const Entry& e : kEntries)
        if (!strcmp(e.name, name)) {
            Launcher* l = PyObject_GC_New(Launcher, &LauncherType);
            if (!l) return nullptr;
            l->dict = nullptr;
            l->weakrefs = nullptr;
            l->fallback = fallback;
            l->failed = failed;
            Py_INCREF(fallback);
            Py_INCREF(failed);
            l->entry = &e;
            for (int i = 0; i < kMaxParams; ++i) l->names[i] = i < e.n_params ? PyUnicode_InternFromString(e.params[i]) : nullptr;
            l->vectorcall = launcher_call;
            PyObject_GC_Track((PyObject*)l);
            return (PyObject*)l;
        }
    Py_RETURN_NONE;
}

// Objects, the attributes of the instances of Python classes among them, and where and how every tensor of these lies in
// memory, as a row of numbers: written to `out`, or compared with an earlier row as it goes.
struct Row {
    std::string* out;
    const char *at, *end;
    bool put(int64_t v) {
        if (out) {
            out->append((const char*)&v, sizeof v);
            return true;
        }
        if (at == end || memcmp(at, &v, sizeof v)) return false;
        at += sizeof v;
        return true;
    }
};

// false: another row (or an error is set). `keep` receives the objects, so that none of their identities is given out again.
bool describe(PyObject* o, bool attributes, Row& row, PyObject* keep) {
    if (!row.put((int64_t)(intptr_t)o) || (keep && PyList_Append(keep, o) < 0)) return false;
    if (PyObject_TypeCheck(o, (PyTypeObject*)THPVariableClass)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!row.put(t.has_storage() ? (int64_t)(intptr_t)t.unsafeGetTensorImpl()->unsafe_storage().data() : -1) ||
            !row.put(t.has_storage() ? t.storage_offset() : 0) || !row.put((int64_t)t.scalar_type() << 8 | (uint8_t)t.device().index()) || !row.put(t.dim())) return false;
        for (int64_t v : t.sizes())
            if (!row.put(v)) return false;
        for (int64_t v : t.strides())
            if (!row.put(v)) return false;
        return true;
    }
    if (!attributes || !PyType_HasFeature(Py_TYPE(o), Py_TPFLAGS_HEAPTYPE)) return true;
    PyObject* d = PyObject_GenericGetDict(o, nullptr);
    if (!d) {                                            // an instance without attributes of its own
        PyErr_Clear();
        return true;
    }
    bool ok = row.put(PyDict_GET_SIZE(d));
    Py_ssize_t pos = 0;
    PyObject *key, *value;
    while (ok && PyDict_Next(d, &pos, &key, &value)) ok = row.put((int64_t)(intptr_t)key) && describe(value, false, row, keep);
    Py_DECREF(d);
    return ok;
}

bool describe_all(PyObject* objects, Row& row, PyObject* keep) {
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(objects); ++i)
        if (!describe(PyTuple_GET_ITEM(objects, i), true, row, keep)) return false;
    return true;
}

// snapshot(objects, keep) -> the row as bytes; the list `keep` receives the objects
PyObject* snapshot(PyObject*, PyObject* args) {
    PyObject *objects, *keep;
    if (!PyArg_ParseTuple(args, "O!O!", &PyTuple_Type, &objects, &PyList_Type, &keep)) return nullptr;
    try {
        std::string out;
        Row row{&out, nullptr, nullptr};
        if (!describe_all(objects, row, keep)) return nullptr;
        return PyBytes_FromStringAndSize(out.data(), (Py_ssize_t)out.size());
    } catch (const std::exception& e) {
        return PyErr_Format(PyExc_RuntimeError, "%s", e.what());
    }
}

// unchanged(objects, row) -> True while nothing was replaced or moved since the snapshot (whose objects live)
PyObject* unchanged(PyObject*, PyObject* args) {
    PyObject *objects, *bytes;
    if (!PyArg_ParseTuple(args, "O!O!", &PyTuple_Type, &objects, &PyBytes_Type, &bytes)) return nullptr;
    try {
        const char* p = PyBytes_AS_STRING(bytes);
        Row row{nullptr, p, p + PyBytes_GET_SIZE(bytes)};
        return PyBool_FromLong(describe_all(objects, row, nullptr) && row.at == row.end);
    } catch (const std::exception& e) {
        return PyErr_Format(PyExc_RuntimeError, "%s", e.what());
    }
}

PyMethodDef methods[] = {{"launcher", make_launcher, METH_VARARGS, nullptr}, {"snapshot", snapshot, METH_VARARGS, nullptr}, {"unchanged", unchanged, METH_VARARGS, nullptr}, {}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__host(void) {
    LauncherType.tp_name = "paper_2512_20861_amd._host.Launcher";
    LauncherType.tp_basicsize = sizeof(Launcher);
    LauncherType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL | Py_TPFLAGS_HAVE_GC;
    LauncherType.tp_dealloc = launcher_dealloc;
    LauncherType.tp_traverse = launcher_traverse;
    LauncherType.tp_dictoffset = offsetof(Launcher, dict);
    LauncherType.tp_getset = launcher_getset;
    LauncherType.tp_methods = launcher_methods;
    LauncherType.tp_weaklistoffset = offsetof(Launcher, weakrefs);
    LauncherType.tp_vectorcall_offset = offsetof(Launcher, vectorcall);
    LauncherType.tp_call = PyVectorcall_Call;
    if (PyType_Ready(&LauncherType) < 0) return nullptr;
    return PyModule_Create(&module);
}
