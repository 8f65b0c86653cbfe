// Argument marshalling of the Python binding in native code: a CPython module beside libqsdp.so that turns tensors and
// numbers into a call of the C ABI. A call over a few 100,000 elements is bound by what happens on the host. In a
// loop, with the checks and the conversions in Python and ctypes / here: fused step over 2^16 parameters 7.5 / 5.3 us,
// encoder 7.9 / 4.7, decoder 7.8 / 4.5, receive side 12.1 / 6.6; about 2.7 us of each is the launch.
//
// Only what is common is done here: plain tensors, arguments of the expected kinds, the tensor's device the current
// one. For anything else the caller's Python function of the same purpose is called with the same arguments, and its
// result or exception is the answer, so that what is accepted, refused and raised stays in one place.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <hip/hip_runtime_api.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/autograd/python_variable.h>

#include <tuple>
#include <utility>

#include "../../include/qsdp.h"

namespace {

// The Python functions for everything else (see attach), and the binding's namespace: the stream is asked for through
// its name `_raw_stream`.
PyObject *is_in_python, *rows_in_python, *packed_in_python, *rows_ok_in_python, *outputs_in_python, *launch_in_python,
    *devices_in_python, *names;
PyObject *raw_stream_name, *segments_name, *device_name;

bool plain_tensor(PyObject* o) { return THPVariable_CheckExact(o); }

// ---- one argument of the C ABI -----------------------------------------------------------------------------------
// As ctypes converts them, where it does so without an error: integers modulo 2^64, floats from any number, pointers
// from None, an address or (here) a tensor. False: left to Python.
bool convert(PyObject* o, uint64_t& out) {
    if (!PyLong_Check(o)) return false;
    out = PyLong_AsUnsignedLongLongMask(o);
    return true;
}
bool convert(PyObject* o, uint32_t& out) {
    uint64_t v;
    if (!convert(o, v)) return false;
    out = (uint32_t)v;
    return true;
}
bool convert(PyObject* o, int& out) {
    uint64_t v;
    if (!convert(o, v)) return false;
    out = (int)(uint32_t)v;
    return true;
}
bool convert(PyObject* o, qsdp_dtype& out) {
    int v;
    if (!convert(o, v)) return false;
    out = (qsdp_dtype)v;
    return true;
}
bool convert(PyObject* o, float& out) {
    if (PyFloat_Check(o)) out = (float)PyFloat_AS_DOUBLE(o);
    else if (PyLong_Check(o)) out = (float)PyLong_AsDouble(o);
    else return false;
    return !PyErr_Occurred();
}
template <class T>
bool convert(PyObject* o, T*& out) {
    if (o == Py_None) {
        out = nullptr;
        return true;
    }
    if (plain_tensor(o)) {
        out = static_cast<T*>(const_cast<void*>(static_cast<const void*>(THPVariable_Unpack(o).data_ptr())));
        return true;
    }
    uint64_t v;
    if (!convert(o, v)) return false;
    out = reinterpret_cast<T*>((uintptr_t)v);
    return true;
}

// ---- the entry points ----------------------------------------------------------------------------------------------
template <class... A, size_t... I>
bool call(int (*entry)(A...), PyObject* const* args, void* stream, int* status, std::index_sequence<I...>) {
    std::tuple<A...> values;
    std::get<sizeof...(A) - 1>(values) = stream;
    if (!(convert(args[I], std::get<I>(values)) && ...)) return false;
    Py_BEGIN_ALLOW_THREADS
    *status = std::apply(entry, values);
    Py_END_ALLOW_THREADS
    return true;
}

struct Entry {
    const char* name;
    int nargs;  // without the stream
    bool (*call)(PyObject* const* args, void* stream, int* status);
};

template <class F>
struct Arity;
template <class... A>
struct Arity<int (*)(A...)> {
    static constexpr size_t n = sizeof...(A);
};

template <auto ENTRY>
constexpr Entry entry(const char* name) {
    constexpr size_t n = Arity<decltype(ENTRY)>::n;
    return {name, (int)n - 1, [](PyObject* const* args, void* stream, int* status) {
                return call(ENTRY, args, stream, status, std::make_index_sequence<n - 1>());
            }};
}

// Every entry point that launches work and takes no options block.
#define E(f) entry<&f>(#f)
const Entry entries[] = {
    E(qsdp_quantize_grad), E(qsdp_quantize_grad_ex), E(qsdp_quantize_grad_g16), E(qsdp_quantize_weight),
    E(qsdp_quantize_weight_ex), E(qsdp_dequantize), E(qsdp_fused_step), E(qsdp_fused_step_ex),
    E(qsdp_fused_step_g16), E(qsdp_fused_step_mp), E(qsdp_fused_step_dseed), E(qsdp_fused_step_codes),
    E(qsdp_fused_adamw_step), E(qsdp_fused_adamw_step_mp), E(qsdp_fused_adamw_step_codes), E(qsdp_dequantize_add),
    E(qsdp_dequantize_gathered), E(qsdp_recv_step), E(qsdp_recv_adamw_step), E(qsdp_quantize_levels),
    E(qsdp_quantize_levels_stochastic), E(qsdp_dequantize_levels), E(qsdp_dequantize_levels_gathered),
    E(qsdp_fit_levels), E(qsdp_quantize_grad_segmented), E(qsdp_quantize_weight_segmented),
    E(qsdp_fused_step_segmented), E(qsdp_fused_step_segmented_mp), E(qsdp_dequantize_segmented),
    E(qsdp_fused_adamw_step_segmented), E(qsdp_fused_step_codes_segmented), E(qsdp_recv_step_segmented),
    E(qsdp_recv_adamw_step_segmented), E(qsdp_fit_levels_segmented), E(qsdp_quantize_levels_segmented),
    E(qsdp_dequantize_levels_segmented)};
#undef E

// Call sites name their entry points by literals, which Python interns, so the object itself is compared.
constexpr size_t kEntries = sizeof(entries) / sizeof(entries[0]);
PyObject* entry_names[kEntries];

const Entry* find_entry(PyObject* name) {
    for (size_t i = 0; i < kEntries; ++i)
        if (entry_names[i] == name) return &entries[i];
    return nullptr;
}

// launch(tensor, name, *args): calls the entry point with the current stream of the tensor's device.
PyObject* launch(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    try {
        const Entry* e = nargs >= 2 ? find_entry(args[1]) : nullptr;
        if (e != nullptr && nargs - 2 == e->nargs && plain_tensor(args[0])) {
            const int device = THPVariable_Unpack(args[0]).get_device();
            int current = -1;
            if (device >= 0 && hipGetDevice(&current) == hipSuccess && current == device) {
                PyObject* raw_stream = PyDict_GetItemWithError(names, raw_stream_name);
                PyObject* number = raw_stream ? PyLong_FromLong(device) : nullptr;
                PyObject* handle = number ? PyObject_CallOneArg(raw_stream, number) : nullptr;
                Py_XDECREF(number);
                if (handle == nullptr) {
                    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "the binding has no _raw_stream");
                    return nullptr;
                }
                const uintptr_t stream = (uintptr_t)PyLong_AsUnsignedLongLongMask(handle);
                Py_DECREF(handle);
                int status = QSDP_OK;
                if (!PyErr_Occurred() && e->call(args + 2, reinterpret_cast<void*>(stream), &status)) {
                    if (status == QSDP_OK) Py_RETURN_NONE;
                    PyObject* error = PyDict_GetItemString(names, "QsdpError");  // borrowed
                    PyObject* instance = error ? PyObject_CallFunction(error, "iO", status, args[1]) : nullptr;
                    if (instance != nullptr) {
                        PyErr_SetObject((PyObject*)Py_TYPE(instance), instance);
                        Py_DECREF(instance);
                    }
                    return nullptr;
                }
            }
        }
    } catch (const std::exception&) {
        // Python asks for the same and reports it
    }
    PyErr_Clear();
    return PyObject_Vectorcall(launch_in_python, args, (size_t)nargs, nullptr);
}

bool has_type(PyObject* o, PyObject* dtype, bool rows) {
    if (!plain_tensor(o) || !THPDtype_Check(dtype)) return false;
    try {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda() || t.scalar_type() != reinterpret_cast<THPDtype*>(dtype)->scalar_type) return false;
        return rows ? t.dim() == 2 && (t.size(1) == 1 || t.stride(1) == 1) : t.is_contiguous();
    } catch (const std::exception&) {
        return false;
    }
}

// is(tensor, dtype): nothing if it is a contiguous GPU tensor of that type; is_rows: if its rows are.
PyObject* is_tensor(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs == 2 && has_type(args[0], args[1], false)) Py_RETURN_NONE;
    return PyObject_Vectorcall(is_in_python, args, (size_t)nargs, nullptr);
}

PyObject* is_rows(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs == 2 && has_type(args[0], args[1], true)) Py_RETURN_NONE;
    return PyObject_Vectorcall(rows_in_python, args, (size_t)nargs, nullptr);
}

// step_outputs(wcodes, wmeta, n_saturated): nothing if each is None or a contiguous GPU tensor of its type.
PyObject* step_outputs(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    const at::ScalarType types[3] = {at::kInt, at::kFloat, at::kLong};
    bool ok = nargs == 3;
    for (int i = 0; ok && i < 3; ++i) {
        if (args[i] == Py_None) continue;
        ok = plain_tensor(args[i]);
        try {
            if (ok) {
                const at::Tensor& t = THPVariable_Unpack(args[i]);
                ok = t.is_cuda() && t.scalar_type() == types[i] && t.is_contiguous();
            }
        } catch (const std::exception&) {
            ok = false;
        }
    }
    if (ok) Py_RETURN_NONE;
    return PyObject_Vectorcall(outputs_in_python, args, (size_t)nargs, nullptr);
}

// Whether buffers (None: not asked) hold the codes and the meta of n elements, in every row or in all.
bool holds(PyObject* const* args, bool rows) {
    const bool codes = plain_tensor(args[0]), meta = plain_tensor(args[1]);
    uint64_t n;
    int bits, bucket;
    if ((!codes && args[0] != Py_None) || (!meta && args[1] != Py_None) || !convert(args[2], n) ||
        !convert(args[3], bits) || !convert(args[4], bucket))
        return false;
    try {
        auto enough = [&](PyObject* o, size_t bytes) {
            const at::Tensor& t = THPVariable_Unpack(o);
            return (uint64_t)(rows ? t.size(1) : t.numel()) >= bytes / 4;
        };
        return (!codes || enough(args[0], qsdp_codes_bytes(n, bits, bucket))) &&
               (!meta || enough(args[1], qsdp_meta_bytes(n, bucket)));
    } catch (const std::exception&) {
        return false;
    }
}

// packed_ok, rows_ok(codes, meta, n, bits, bucket): nothing if the packed buffers, or every row of them, hold n elements.
PyObject* packed_ok(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs == 5 && ((args[0] == Py_None && args[1] == Py_None) || holds(args, false))) Py_RETURN_NONE;
    return PyObject_Vectorcall(packed_in_python, args, (size_t)nargs, nullptr);
}

PyObject* rows_ok(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs == 5 && args[0] != Py_None && args[1] != Py_None && holds(args, true)) Py_RETURN_NONE;
    return PyObject_Vectorcall(rows_ok_in_python, args, (size_t)nargs, nullptr);
}

// Numbers and None hold no tensor. (Subclasses of numbers neither, but they are Python's to ask.)
bool plain_value(PyObject* o) {
    return o == Py_None || PyLong_CheckExact(o) || PyFloat_CheckExact(o) || PyBool_Check(o);
}

// Whether o is a value, or a tensor or segment table on the device of those before it (none yet: -2).
bool same_device(PyObject* o, int& device) {
    if (plain_value(o)) return true;
    if (!plain_tensor(o)) {  // a table's tensor is its attribute `device`
        if ((PyObject*)Py_TYPE(o) != PyDict_GetItem(names, segments_name)) return false;
        PyObject* table = PyObject_GetAttr(o, device_name);
        if (table == nullptr) PyErr_Clear();
        const bool ok = table != nullptr && plain_tensor(table) && same_device(table, device);
        Py_XDECREF(table);
        return ok;
    }
    try {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda()) return false;
        const int here = t.get_device();
        if (device == -2) device = here;
        return here == device;
    } catch (const std::exception&) {
        return false;
    }
}

// devices_ok(name, args, kwargs): nothing if all tensors among the arguments are on one GPU. In a loop 1.1-1.5 us less
// than in Python (fused step over 2^20 parameters 6.0 -> 4.5 us, encoder of 2^18 values 5.6 -> 4.5, gathered layer 6.4
// -> 5.3, encoder and decoder 10.9 -> 8.9; calls over tensors, whose table is looked at too, 5.4-6.0 -> 4.3-4.7).
PyObject* devices_ok(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs == 3 && PyTuple_CheckExact(args[1]) && PyDict_CheckExact(args[2])) {
        int device = -2;
        bool ok = true;
        for (Py_ssize_t i = 0; ok && i < PyTuple_GET_SIZE(args[1]); ++i)
            ok = same_device(PyTuple_GET_ITEM(args[1], i), device);
        PyObject *key, *value;
        for (Py_ssize_t at = 0; ok && PyDict_Next(args[2], &at, &key, &value);) ok = same_device(value, device);
        if (ok) Py_RETURN_NONE;
    }
    return PyObject_Vectorcall(devices_in_python, args, (size_t)nargs, nullptr);
}

// attach(names, is, is_rows, packed_ok, rows_ok, step_outputs, launch, devices_ok): the binding's namespace and its
// functions for what is not common.
PyObject* attach(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 8 || !PyDict_Check(args[0])) {
        PyErr_SetString(PyExc_TypeError,
                        "attach(namespace, is, is_rows, packed_ok, rows_ok, step_outputs, launch, devices_ok)");
        return nullptr;
    }
    PyObject** const held[8] = {&names, &is_in_python, &rows_in_python, &packed_in_python, &rows_ok_in_python,
                                &outputs_in_python, &launch_in_python, &devices_in_python};
    for (int i = 0; i < 8; ++i) {
        Py_INCREF(args[i]);
        Py_XSETREF(*held[i], args[i]);
    }
    Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}
PyMethodDef methods[] = {method<attach>("attach"), method<is_tensor>("is"), method<is_rows>("is_rows"),
                         method<packed_ok>("packed_ok"), method<rows_ok>("rows_ok"),
                         method<step_outputs>("step_outputs"), method<launch>("launch"),
                         method<devices_ok>("devices_ok"), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_marshal", "Argument marshalling of the binding.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
    raw_stream_name = PyUnicode_InternFromString("_raw_stream");
    segments_name = PyUnicode_InternFromString("Segments");
    device_name = PyUnicode_InternFromString("device");
    if (raw_stream_name == nullptr || segments_name == nullptr || device_name == nullptr) return nullptr;
    for (size_t i = 0; i < kEntries; ++i) {
        entry_names[i] = PyUnicode_InternFromString(entries[i].name);
        if (entry_names[i] == nullptr) return nullptr;
    }
    PyObject* module = PyModule_Create(&module_def);
    // The layouts compiled in are those of this torch; the binding compares before it uses anything else.
    if (module != nullptr && PyModule_AddStringConstant(module, "torch_version", QSDP_TORCH_VERSION) != 0) {
        Py_DECREF(module);
        return nullptr;
    }
    return module;
}
