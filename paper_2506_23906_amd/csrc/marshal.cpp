// The argument marshalling of binding.py for the calls that a program makes over and over, as a CPython extension: tensors to
// pointers, the current stream, the call of the C entry point.  A call on a short vector takes the GPU three microseconds; with
// properties asked for one by one in Python and ctypes converting ten arguments, the host took 4.7 to issue it (segmented scan of
// 3000 values; see binding.py for what it takes now).
// Every function returns the status of the entry point, or None for a call it leaves to binding.py: arguments left out, types it does
// not know, subclasses of Tensor, tensors that are not contiguous GPU memory (binding.py raises what it raises for those).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "mmvseg.h"

namespace {

struct {
    decltype(&mmv_segscan) segscan;
    decltype(&mmv_segsum) segsum;
    decltype(&mmv_scan) scan;
    decltype(&mmv_compress) compress;
    decltype(&mmv_spmv_coo) spmv_coo, spmv_coo_run;
    decltype(&mmv_spmv_csr) spmv_csr, spmv_csr_run;
} g_entry;

struct LeftToPython {};   // thrown and caught in here

struct Array {
    void *ptr;
    uint64_t numel;
    at::ScalarType type;
};
Array array(PyObject *o) {
    if (!THPVariable_CheckExact(o)) throw LeftToPython();
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) throw LeftToPython();
    return {t.data_ptr(), (uint64_t)t.numel(), t.scalar_type()};
}
uint64_t number(PyObject *o) {
    if (!PyLong_CheckExact(o)) throw LeftToPython();
    return PyLong_AsUnsignedLongLongMask(o);
}
mmv_dtype value_type(const Array &a) {
    switch (a.type) {
        case at::kFloat: return MMV_F32_F32;
        case at::kHalf: return MMV_F16_F32;
        case at::kBFloat16: return MMV_BF16_F32;
        case at::kChar: return MMV_I8_I32;
        case at::kByte: return MMV_U8_XOR;
        default: throw LeftToPython();
    }
}
mmv_flag_fmt flag_format(const Array &a) {
    if (a.type == at::kByte) return MMV_FLAGS_U8;
    if (a.type == at::kInt) return MMV_FLAGS_PACKED32;
    throw LeftToPython();
}
mmv_variant variant(PyObject *o) {
    if (PyUnicode_CheckExact(o)) {
        if (PyUnicode_CompareWithASCIIString(o, "mfma") == 0) return MMV_VARIANT_MFMA;
        if (PyUnicode_CompareWithASCIIString(o, "shuffle") == 0) return MMV_VARIANT_SHUFFLE;
    }
    throw LeftToPython();
}
void *stream(PyObject *o) {   // (None: the current one of the current device)
    if (o != Py_None) throw LeftToPython();
    return (void *)c10::hip::getCurrentHIPStream().stream();
}

template <typename Body> PyObject *guarded(Py_ssize_t got, Py_ssize_t want, Body body) {
    if (got != want) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    try {
        return PyLong_FromLong((long)body());
    } catch (...) {   // (also what torch throws for tensors without memory of their own)
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}
struct WithoutGil {
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

// segscan(x, flags, n, z, variant, ws, stream)
PyObject *segscan(PyObject *, PyObject *const *a, Py_ssize_t count) {
    return guarded(count, 7, [&] {
        const Array x = array(a[0]), f = array(a[1]), z = array(a[3]), ws = array(a[5]);
        const uint64_t n = a[2] == Py_None ? x.numel : number(a[2]);
        const mmv_dtype dt = value_type(x);
        const mmv_flag_fmt ff = flag_format(f);
        const mmv_variant v = variant(a[4]);
        void *const s = stream(a[6]);
        WithoutGil free;
        return g_entry.segscan(x.ptr, f.ptr, n, z.ptr, dt, ff, v, ws.ptr, ws.numel, s);
    });
}
// segsum(x, flags, n, out, nseg, variant, ws, stream)
PyObject *segsum(PyObject *, PyObject *const *a, Py_ssize_t count) {
    return guarded(count, 8, [&] {
        const Array x = array(a[0]), f = array(a[1]), out = array(a[3]), nseg = array(a[4]), ws = array(a[6]);
        const uint64_t n = a[2] == Py_None ? x.numel : number(a[2]);
        const mmv_dtype dt = value_type(x);
        const mmv_flag_fmt ff = flag_format(f);
        const mmv_variant v = variant(a[5]);
        void *const s = stream(a[7]);
        WithoutGil free;
        return g_entry.segsum(x.ptr, f.ptr, n, out.ptr, out.numel, (uint64_t *)nseg.ptr, dt, ff, v, ws.ptr, ws.numel, s);
    });
}
// scan(x, n, z, variant, ws, stream)
PyObject *scan(PyObject *, PyObject *const *a, Py_ssize_t count) {
    return guarded(count, 6, [&] {
        const Array x = array(a[0]), z = array(a[2]), ws = array(a[4]);
        const uint64_t n = a[1] == Py_None ? x.numel : number(a[1]);
        const mmv_dtype dt = value_type(x);
        const mmv_variant v = variant(a[3]);
        void *const s = stream(a[5]);
        WithoutGil free;
        return g_entry.scan(x.ptr, n, z.ptr, dt, v, ws.ptr, ws.numel, s);
    });
}
// compress(x, mask, n, out, count, ws, stream)
PyObject *compress(PyObject *, PyObject *const *a, Py_ssize_t args) {
    return guarded(args, 7, [&] {
        Array x = {};
        if (a[0] != Py_None) {
            x = array(a[0]);
            if (c10::elementSize(x.type) != 4) throw LeftToPython();
        }
        const Array mask = array(a[1]), out = array(a[3]), count = array(a[4]), ws = array(a[5]);
        const uint64_t n = number(a[2]);
        const mmv_flag_fmt ff = flag_format(mask);
        void *const s = stream(a[6]);
        WithoutGil free;
        return g_entry.compress(x.ptr, mask.ptr, n, out.ptr, out.numel, (uint64_t *)count.ptr, ff, ws.ptr, ws.numel, s);
    });
}
// ...(n_rows, n_cols, nnz, row or rowptr, col, val, x, y, variant, ws, stream)
template <typename Entry> PyObject *spmv(Entry entry, PyObject *const *a, Py_ssize_t args) {
    return guarded(args, 11, [&] {
        const uint64_t n_rows = number(a[0]), n_cols = number(a[1]);
        const Array row = array(a[3]), col = array(a[4]), val = array(a[5]), x = array(a[6]), y = array(a[7]), ws = array(a[9]);
        const uint64_t nnz = a[2] == Py_None ? val.numel : number(a[2]);
        const mmv_variant v = variant(a[8]);
        void *const s = stream(a[10]);
        WithoutGil free;
        return entry(n_rows, n_cols, nnz, (const int32_t *)row.ptr, (const int32_t *)col.ptr, (const float *)val.ptr, (const float *)x.ptr,
                     (float *)y.ptr, v, ws.ptr, ws.numel, s);
    });
}
PyObject *spmv_coo(PyObject *, PyObject *const *a, Py_ssize_t n) { return spmv(g_entry.spmv_coo, a, n); }
PyObject *spmv_csr(PyObject *, PyObject *const *a, Py_ssize_t n) { return spmv(g_entry.spmv_csr, a, n); }
PyObject *spmv_coo_run(PyObject *, PyObject *const *a, Py_ssize_t n) { return spmv(g_entry.spmv_coo_run, a, n); }
PyObject *spmv_csr_run(PyObject *, PyObject *const *a, Py_ssize_t n) { return spmv(g_entry.spmv_csr_run, a, n); }

// bind(addresses of mmv_segscan, mmv_segsum, mmv_scan, mmv_compress, mmv_spmv_coo, mmv_spmv_csr, mmv_spmv_coo_run, mmv_spmv_csr_run)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t count) {
    void *p[8];
    if (count != 8) {
        PyErr_SetString(PyExc_TypeError, "bind takes eight addresses");
        return nullptr;
    }
    for (int i = 0; i < 8; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i] && PyErr_Occurred()) return nullptr;
    }
    g_entry = {(decltype(&mmv_segscan))p[0], (decltype(&mmv_segsum))p[1], (decltype(&mmv_scan))p[2], (decltype(&mmv_compress))p[3],
               (decltype(&mmv_spmv_coo))p[4], (decltype(&mmv_spmv_coo))p[6], (decltype(&mmv_spmv_csr))p[5], (decltype(&mmv_spmv_csr))p[7]};
    Py_RETURN_NONE;
}

#define MMV_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {MMV_METHOD(bind),     MMV_METHOD(segscan),      MMV_METHOD(segsum),       MMV_METHOD(scan),
                           MMV_METHOD(compress), MMV_METHOD(spmv_coo),     MMV_METHOD(spmv_csr),     MMV_METHOD(spmv_coo_run),
                           MMV_METHOD(spmv_csr_run), {nullptr, nullptr, 0, nullptr}};
#undef MMV_METHOD
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", "Argument marshalling of the calls of libmmvseg.so.", -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
    PyObject *m = PyModule_Create(&g_module);
    if (m && PyModule_AddStringConstant(m, "torch_version", MMV_TORCH_VERSION) < 0) Py_CLEAR(m);   // (binding.py uses it with this one only)
    return m;
}
