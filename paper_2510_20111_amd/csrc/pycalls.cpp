// The Python calls that a training program makes for every layer of every step, without the interpreter's share of
// them: a Call object takes the arguments of one binding function, converts them and calls the C entry point.  What it
// does not recognise (other types, missing or unknown arguments, more than 512 pointers in lists) goes to the
// binding function itself, which converts or refuses it as it always did; this is seen before any tensor is asked for its
// address, so that no work is done twice.
//
// A 64 k element call costs the binding function 0.45 us in the interpreter and ctypes 0.5 us, of 3.7 us in all; this
// takes 0.15 us.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>

#include <cstddef>
#include <cstdint>
#include <cstring>
#include <initializer_list>

#include "hzp.h"

namespace {

constexpr int kMostArgs = 13;
constexpr Py_ssize_t kMostListed = 512;         // pointers of lists and tuples in one call; longer ones go the other way

enum Kind {
    kPlan,          // object whose `handle` is a c_void_p
    kU32, kI32,
    kFloat,
    kFlag,          // True or False
    kPointers,      // ctypes array, or list or tuple of addresses
    kAddress,       // None, an integer or an object with data_ptr()
    kHyper,         // the binding's AdamW
    kStream,        // an integer, an object with cuda_stream, or None: torch's current stream
    kCount,         // an integer, or None: the length of the first kPointers argument
};

struct Arg {
    const char *name;
    Kind kind;
    enum { kRequired, kNone, kZero, kMayBeNone } if_missing;    // kMayBeNone: required, and None is a null pointer
};

struct Value {
    uint64_t word;      // numbers, addresses
    float real;
    Py_ssize_t length;  // of kPointers
};

struct Function {
    const char *name;
    int n_args;
    Arg args[kMostArgs];
    hzp_status_t (*call)(void *fn, const Value *v);
};

template <class T>
T ptr(const Value &v) { return reinterpret_cast<T>(static_cast<uintptr_t>(v.word)); }
uint32_t u32(const Value &v) { return (uint32_t)v.word; }
typedef const hzp_plan_t *plan_p;
typedef const void *const *sources_p;
typedef void *const *outputs_p;
typedef float *const *floats_p;

const Function kFunctions[] = {
    {"hzp_reduce_shard", 12,
     {{"plan", kPlan}, {"layer", kU32}, {"cls", kU32}, {"level", kI32}, {"rank", kU32}, {"grad_slices", kPointers}, {"scale", kFloat},
      {"accumulate", kFlag}, {"out_f32", kAddress}, {"stream", kStream, Arg::kNone}, {"R", kCount, Arg::kNone}, {"grad_dtype", kU32, Arg::kZero}},
     [](void *fn, const Value *v) {
         return reinterpret_cast<decltype(&hzp_reduce_shard)>(fn)(ptr<plan_p>(v[0]), u32(v[1]), u32(v[2]), (int)v[3].word, u32(v[4]), ptr<sources_p>(v[5]),
                                                                  u32(v[10]), u32(v[11]), v[6].real, (int)v[7].word, ptr<float *>(v[8]),
                                                                  ptr<hipStream_t>(v[9]));
     }},
    {"hzp_adamw_shard", 13,
     {{"plan", kPlan}, {"layer_begin", kU32}, {"layer_end", kU32}, {"cls", kU32}, {"rank", kU32}, {"hyper", kHyper}, {"grad_slices", kPointers},
      {"R", kU32}, {"master", kPointers}, {"m", kPointers}, {"v", kPointers}, {"param_out", kPointers, Arg::kMayBeNone}, {"stream", kStream, Arg::kNone}},
     [](void *fn, const Value *v) {
         return reinterpret_cast<decltype(&hzp_adamw_shard)>(fn)(ptr<plan_p>(v[0]), u32(v[1]), u32(v[2]), u32(v[3]), u32(v[4]),
                                                                 ptr<const hzp_adamw_t *>(v[5]), ptr<sources_p>(v[6]), u32(v[7]), ptr<floats_p>(v[8]),
                                                                 ptr<floats_p>(v[9]), ptr<floats_p>(v[10]), ptr<outputs_p>(v[11]), ptr<hipStream_t>(v[12]));
     }},
    {"hzp_adamw_shard_dev", 13,
     {{"plan", kPlan}, {"layer_begin", kU32}, {"layer_end", kU32}, {"cls", kU32}, {"rank", kU32}, {"scalars", kAddress}, {"grad_slices", kPointers},
      {"R", kU32}, {"master", kPointers}, {"m", kPointers}, {"v", kPointers}, {"param_out", kPointers, Arg::kMayBeNone}, {"stream", kStream, Arg::kNone}},
     [](void *fn, const Value *v) {
         return reinterpret_cast<decltype(&hzp_adamw_shard_dev)>(fn)(ptr<plan_p>(v[0]), u32(v[1]), u32(v[2]), u32(v[3]), u32(v[4]),
                                                                     ptr<const hzp_adamw_scalars_t *>(v[5]), ptr<sources_p>(v[6]), u32(v[7]),
                                                                     ptr<floats_p>(v[8]), ptr<floats_p>(v[9]), ptr<floats_p>(v[10]),
                                                                     ptr<outputs_p>(v[11]), ptr<hipStream_t>(v[12]));
     }},
    {"hzp_gather_layer", 9,
     {{"plan", kPlan}, {"layer", kU32}, {"cls", kU32}, {"level", kI32}, {"shard_ptrs", kPointers}, {"bucket_out", kAddress, Arg::kNone},
      {"tensor_out", kPointers, Arg::kNone}, {"stream", kStream, Arg::kNone}, {"n_shards", kCount, Arg::kNone}},
     [](void *fn, const Value *v) {
         return reinterpret_cast<decltype(&hzp_gather_layer)>(fn)(ptr<plan_p>(v[0]), u32(v[1]), u32(v[2]), (int)v[3].word, ptr<sources_p>(v[4]), u32(v[8]),
                                                                  ptr<void *>(v[5]), ptr<outputs_p>(v[6]), ptr<hipStream_t>(v[7]));
     }},
    {"hzp_gather_layer_static", 7,
     {{"plan", kPlan}, {"layer", kU32}, {"cls", kU32}, {"shard_ptrs", kPointers}, {"tensor_out", kPointers, Arg::kMayBeNone},
      {"stream", kStream, Arg::kNone}, {"n_shards", kCount, Arg::kNone}},
     [](void *fn, const Value *v) {
         return reinterpret_cast<decltype(&hzp_gather_layer_static)>(fn)(ptr<plan_p>(v[0]), u32(v[1]), u32(v[2]), ptr<sources_p>(v[3]), u32(v[6]),
                                                                         ptr<outputs_p>(v[4]), ptr<hipStream_t>(v[5]));
     }},
    {"hzp_gather_shard", 8,
     {{"plan", kPlan}, {"layer", kU32}, {"cls", kU32}, {"j", kU32}, {"owner_ptrs", kPointers}, {"shard_out", kAddress},
      {"stream", kStream, Arg::kNone}, {"n_owners", kCount, Arg::kNone}},
     [](void *fn, const Value *v) {
         return reinterpret_cast<decltype(&hzp_gather_shard)>(fn)(ptr<plan_p>(v[0]), u32(v[1]), u32(v[2]), u32(v[3]), ptr<sources_p>(v[4]), u32(v[7]),
                                                                  ptr<void *>(v[5]), ptr<hipStream_t>(v[6]));
     }},
    {"hzp_gather_layers", 9,
     {{"plan", kPlan}, {"layer_begin", kU32}, {"layer_end", kU32}, {"cls", kU32}, {"level", kI32}, {"shard_ptrs", kPointers}, {"n_shards", kU32},
      {"bucket_out", kPointers}, {"stream", kStream, Arg::kNone}},
     [](void *fn, const Value *v) {
         return reinterpret_cast<decltype(&hzp_gather_layers)>(fn)(ptr<plan_p>(v[0]), u32(v[1]), u32(v[2]), u32(v[3]), (int)v[4].word, ptr<sources_p>(v[5]),
                                                                   u32(v[6]), ptr<outputs_p>(v[7]), ptr<hipStream_t>(v[8]));
     }},
    {"hzp_gather_tensor", 6,
     {{"plan", kPlan}, {"tensor_id", kU32}, {"shard_ptrs", kPointers}, {"tensor_out", kAddress}, {"stream", kStream, Arg::kNone},
      {"n_shards", kCount, Arg::kNone}},
     [](void *fn, const Value *v) {
         return reinterpret_cast<decltype(&hzp_gather_tensor)>(fn)(ptr<plan_p>(v[0]), u32(v[1]), ptr<sources_p>(v[2]), u32(v[5]), ptr<void *>(v[3]),
                                                                   ptr<hipStream_t>(v[4]));
     }},
};

struct CallObject {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    const Function *function;
    void *entry;                    // the C entry point
    PyObject *names;                // tuple of interned argument names
    PyObject *otherwise;            // the binding function
    PyObject *check;                // raises where a status is not HZP_OK
    PyObject *array, *void_p, *hyper;   // ctypes.Array, ctypes.c_void_p, the binding's AdamW
    PyObject *current_stream;       // what gives the stream where none is given (or null: the binding function does)
    PyObject *code, *defaults;      // the binding function's when this was made
    PyObject *weak;                 // weak references
};

PyObject *name_handle, *name_data_ptr, *name_cuda_stream;      // interned

// Address of a ctypes object's memory (which stays where it is while the caller holds the object).
bool memory_of(PyObject *o, void **address)
{
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return false;
    }
    *address = view.buf;
    PyBuffer_Release(&view);
    return true;
}

// The functions from here to convert_all return false where the binding function has to look at the arguments, and also,
// with the error set, where an argument's own code (data_ptr(), cuda_stream) raised: then that is the call's error.
bool word_of(PyObject *o, uint64_t most, uint64_t *out)
{
    if (!PyLong_CheckExact(o)) return false;
    *out = PyLong_AsUnsignedLongLong(o);
    if (*out == (uint64_t)-1 && PyErr_Occurred()) {     // negative or too long
        PyErr_Clear();
        return false;
    }
    return *out <= most;
}

bool address_of(PyObject *o, uint64_t *out)
{
    if (o == Py_None) {
        *out = 0;
        return true;
    }
    if (PyLong_Check(o)) return word_of(o, ~0ull, out);
    PyObject *const x = PyObject_CallMethodNoArgs(o, name_data_ptr);
    if (!x) return false;
    const bool ok = word_of(x, ~0ull, out);
    Py_DECREF(x);
    return ok;
}

// Converts an argument that runs no code of its own; of the others it only looks at the type, and adds up the lengths of lists.
bool look_at(const CallObject *self, const Arg &arg, PyObject *o, Value *v, Py_ssize_t *n_listed)
{
    switch (arg.kind) {
    case kPlan: {
        PyObject *const handle = PyObject_GetAttr(o, name_handle);
        if (!handle) {
            if (PyErr_ExceptionMatches(PyExc_AttributeError)) PyErr_Clear();
            return false;
        }
        void *at = nullptr;
        const bool ok = (PyObject *)Py_TYPE(handle) == self->void_p && memory_of(handle, &at);
        if (ok) std::memcpy(&v->word, at, sizeof v->word);
        Py_DECREF(handle);
        return ok;
    }
    case kU32: return word_of(o, 0xFFFFFFFFull, &v->word);
    case kI32: return word_of(o, 0x7FFFFFFFull, &v->word);
    case kCount: return word_of(o, 0xFFFFFFFFull, &v->word);
    case kFloat:
        if (!PyFloat_CheckExact(o)) return false;
        v->real = (float)PyFloat_AS_DOUBLE(o);
        return true;
    case kFlag:
        v->word = o == Py_True;
        return o == Py_True || o == Py_False;
    case kHyper: {
        void *at = nullptr;
        if ((PyObject *)Py_TYPE(o) != self->hyper || !memory_of(o, &at)) return false;
        v->word = reinterpret_cast<uintptr_t>(at);
        return true;
    }
    case kPointers:
        if (PyObject_TypeCheck(o, (PyTypeObject *)self->array)) return true;
        if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return false;
        *n_listed += PySequence_Fast_GET_SIZE(o);
        return *n_listed <= kMostListed;
    case kAddress:
    case kStream: return !PyLong_Check(o) || word_of(o, ~0ull, &v->word);
    }
    return false;
}

// Converts an argument that may run code of its own; `listed` has room for the pointers of lists.
bool ask(const CallObject *self, const Arg &arg, PyObject *o, Value *v, void **listed, Py_ssize_t *n_listed)
{
    switch (arg.kind) {
    case kAddress: return address_of(o, &v->word);
    case kStream: {
        if (PyLong_Check(o)) return true;
        PyObject *const x = o == Py_None ? PyObject_CallOneArg(self->current_stream, o) : PyObject_GetAttr(o, name_cuda_stream);
        if (!x) return false;
        const bool ok = word_of(x, ~0ull, &v->word);
        Py_DECREF(x);
        return ok;
    }
    case kPointers:
        if (PyObject_TypeCheck(o, (PyTypeObject *)self->array)) {
            void *at = nullptr;
            if (!memory_of(o, &at)) return false;
            v->word = reinterpret_cast<uintptr_t>(at);
            v->length = PyObject_Size(o);
            return v->length >= 0;
        } else {
            void **const out = listed + *n_listed;
            v->word = reinterpret_cast<uintptr_t>(out);
            // (an element's data_ptr() may run Python code: the size is asked for again each time)
            for (v->length = 0; v->length < PySequence_Fast_GET_SIZE(o); ++v->length) {
                if (*n_listed == kMostListed) return false;
                PyObject *const item = PySequence_Fast_GET_ITEM(o, v->length);
                Py_INCREF(item);
                uint64_t word = 0;
                const bool ok = address_of(item, &word);
                Py_DECREF(item);
                if (!ok) return false;
                listed[(*n_listed)++] = reinterpret_cast<void *>(static_cast<uintptr_t>(word));
            }
            return true;
        }
    default: return true;
    }
}

// Fills the values of all arguments.
bool convert_all(const CallObject *self, PyObject *const *args, Py_ssize_t n, PyObject *kwnames, Value *v, void **listed)
{
    const Function &f = *self->function;
    if (n > f.n_args) return false;
    PyObject *given[kMostArgs] = {};
    for (Py_ssize_t i = 0; i < n; ++i) given[i] = args[i];
    const Py_ssize_t n_kw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < n_kw; ++k) {
        PyObject *const name = PyTuple_GET_ITEM(kwnames, k);
        int at = 0;                                 // names in calls are interned, as these are
        while (at < f.n_args && PyTuple_GET_ITEM(self->names, at) != name) ++at;
        if (at == f.n_args || given[at]) return false;
        given[at] = args[n + k];
    }
    Py_ssize_t n_listed = 0, length = 0;
    bool have_length = false;
    for (int i = 0; i < f.n_args; ++i) {
        const Arg &arg = f.args[i];
        PyObject *&o = given[i];
        v[i] = Value{0, 0.0f, 0};
        if (!o) {
            if (arg.if_missing == Arg::kRequired || arg.if_missing == Arg::kMayBeNone) return false;
            if (arg.if_missing == Arg::kNone) o = Py_None;
        }
        if (arg.kind == kStream && o == Py_None) {
            if (!self->current_stream) return false;
        } else if (o == Py_None && arg.if_missing != Arg::kRequired && arg.if_missing != Arg::kZero) {
            o = nullptr;        // a null pointer, or a count to be filled in below
        } else if (o && !look_at(self, arg, o, &v[i], &n_listed)) {
            return false;
        }
    }
    n_listed = 0;
    for (int i = 0; i < f.n_args; ++i) {            // (in the order in which the binding functions ask)
        const Arg &arg = f.args[i];
        if (given[i] && !ask(self, arg, given[i], &v[i], listed, &n_listed)) return false;
        if (arg.kind == kPointers && !have_length) {
            have_length = true;
            length = v[i].length;
        }
        if (arg.kind == kCount && !given[i]) v[i].word = (uint64_t)length;
    }
    return true;
}

// The binding function is still what this stands for (a program may have given it other defaults or another body).
bool as_made(const CallObject *self)
{
    PyObject *const f = self->otherwise;
    return PyFunction_GET_CODE(f) == self->code && PyFunction_GET_DEFAULTS(f) == self->defaults && !PyFunction_GET_KW_DEFAULTS(f);
}

PyObject *call(PyObject *object, PyObject *const *args, size_t nargsf, PyObject *kwnames)
{
    CallObject *const self = reinterpret_cast<CallObject *>(object);
    Value v[kMostArgs];
    void *listed[kMostListed];
    if (!as_made(self) || !convert_all(self, args, PyVectorcall_NARGS(nargsf), kwnames, v, listed))
        return PyErr_Occurred() ? nullptr : PyObject_Vectorcall(self->otherwise, args, nargsf, kwnames);
    hzp_status_t st;
    Py_BEGIN_ALLOW_THREADS
    st = self->function->call(self->entry, v);
    Py_END_ALLOW_THREADS
    if (st == HZP_OK) Py_RETURN_NONE;
    return PyObject_CallFunction(self->check, "i", (int)st);
}

// Call(name, entry point's address, binding function, check, ctypes.Array, ctypes.c_void_p, AdamW[, function that maps None to the current
// stream's address])
PyObject *make(PyTypeObject *type, PyObject *args, PyObject *)
{
    const char *name;
    unsigned long long entry;
    PyObject *otherwise, *check, *array, *void_p, *hyper, *current_stream = nullptr;
    if (!PyArg_ParseTuple(args, "sKO!OO!O!O!|O", &name, &entry, &PyFunction_Type, &otherwise, &check, &PyType_Type, &array, &PyType_Type, &void_p, &PyType_Type, &hyper,
                          &current_stream))
        return nullptr;
    const Function *function = nullptr;
    for (const Function &f : kFunctions)
        if (!std::strcmp(f.name, name)) function = &f;
    if (!function || !entry) return PyErr_Format(PyExc_ValueError, "no such entry point: %s", name);
    PyObject *const names = PyTuple_New(function->n_args);
    if (!names) return nullptr;
    for (int i = 0; i < function->n_args; ++i) {
        PyObject *const s = PyUnicode_InternFromString(function->args[i].name);
        if (!s) {
            Py_DECREF(names);
            return nullptr;
        }
        PyTuple_SET_ITEM(names, i, s);
    }
    CallObject *const self = reinterpret_cast<CallObject *>(type->tp_alloc(type, 0));
    if (!self) {
        Py_DECREF(names);
        return nullptr;
    }
    self->vectorcall = call;
    self->function = function;
    self->entry = reinterpret_cast<void *>(static_cast<uintptr_t>(entry));
    self->names = names;
    PyObject **const kept[] = {&self->otherwise, &self->check, &self->array, &self->void_p, &self->hyper, &self->code, &self->defaults, &self->current_stream};
    PyObject *const given[] = {otherwise, check, array, void_p, hyper, PyFunction_GET_CODE(otherwise), PyFunction_GET_DEFAULTS(otherwise), current_stream};
    for (int i = 0; i < 8; ++i) {
        Py_XINCREF(given[i]);
        *kept[i] = given[i];
    }
    return reinterpret_cast<PyObject *>(self);
}

void drop(PyObject *object)
{
    CallObject *const self = reinterpret_cast<CallObject *>(object);
    PyTypeObject *const type = Py_TYPE(object);
    if (self->weak) PyObject_ClearWeakRefs(object);
    Py_XDECREF(self->names);
    Py_XDECREF(self->otherwise);
    Py_XDECREF(self->check);
    Py_XDECREF(self->array);
    Py_XDECREF(self->void_p);
    Py_XDECREF(self->hyper);
    Py_XDECREF(self->code);
    Py_XDECREF(self->defaults);
    Py_XDECREF(self->current_stream);
    type->tp_free(object);
    Py_DECREF(type);
}

// To Python the object is the binding function: attributes of all kinds are that function's (its class among them, so that it counts as
// a function), it shows as that function does, becomes a method in a class, and is pickled and copied by its qualified name.
PyObject *attribute(PyObject *object, PyObject *name)
{
    CallObject *const self = reinterpret_cast<CallObject *>(object);
    if (PyUnicode_CompareWithASCIIString(name, "__wrapped__") == 0) {
        Py_INCREF(self->otherwise);
        return self->otherwise;
    }
    for (const char *own : {"__reduce__", "__reduce_ex__", "__get__", "__call__", "__eq__", "__ne__", "__hash__"})
        if (PyUnicode_CompareWithASCIIString(name, own) == 0) return PyObject_GenericGetAttr(object, name);
    return PyObject_GetAttr(self->otherwise, name);
}

int set_attribute(PyObject *object, PyObject *name, PyObject *value)
{
    return PyObject_SetAttr(reinterpret_cast<CallObject *>(object)->otherwise, name, value);
}

PyObject *represent(PyObject *object) { return PyObject_Repr(reinterpret_cast<CallObject *>(object)->otherwise); }

PyObject *bound(PyObject *object, PyObject *instance, PyObject *)
{
    if (instance && instance != Py_None) return PyMethod_New(object, instance);
    Py_INCREF(object);
    return object;
}

PyObject *reduce(PyObject *object, PyObject *)
{
    return PyObject_GetAttrString(reinterpret_cast<CallObject *>(object)->otherwise, "__qualname__");
}

PyMethodDef methods[] = {{"__reduce__", reduce, METH_NOARGS, nullptr}, {nullptr}};
PyMemberDef members[] = {{"__vectorcalloffset__", T_PYSSIZET, offsetof(CallObject, vectorcall), READONLY, nullptr},
                         {"__weaklistoffset__", T_PYSSIZET, offsetof(CallObject, weak), READONLY, nullptr},
                         {nullptr}};
PyType_Slot slots[] = {{Py_tp_new, reinterpret_cast<void *>(make)},
                       {Py_tp_dealloc, reinterpret_cast<void *>(drop)},
                       {Py_tp_call, reinterpret_cast<void *>(PyVectorcall_Call)},
                       {Py_tp_getattro, reinterpret_cast<void *>(attribute)},
                       {Py_tp_setattro, reinterpret_cast<void *>(set_attribute)},
                       {Py_tp_repr, reinterpret_cast<void *>(represent)},
                       {Py_tp_descr_get, reinterpret_cast<void *>(bound)},
                       {Py_tp_methods, methods},
                       {Py_tp_members, members},
                       {0, nullptr}};
PyType_Spec spec = {"_calls.Call", sizeof(CallObject), 0, Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL, slots};
PyModuleDef definition = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls()
{
    name_handle = PyUnicode_InternFromString("handle");
    name_data_ptr = PyUnicode_InternFromString("data_ptr");
    name_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!name_handle || !name_data_ptr || !name_cuda_stream) return nullptr;
    PyObject *const module = PyModule_Create(&definition);
    if (!module) return nullptr;
    PyObject *const type = PyType_FromSpec(&spec);
    if (!type || PyModule_AddObject(module, "Call", type) < 0) {
        Py_XDECREF(type);
        Py_DECREF(module);
        return nullptr;
    }
    return module;
}
