// The binding's tensor views, built in one call: {name: view} over a loaded
// buffer from the sllm_tensor_info table (Sec. 4.1: each tensor's pointer is
// base + offset).
//
// Building the views of a checkpoint of many tensors used to take longer than
// its transfer: per tensor about 0.6 us to decode the table into Python objects
// and 1.1 us for a call of as_strided from Python (4,001 tensors: 6.8 ms,
// against 2.7 ms on the link for their 150 MB).  Here each view is one
// as_strided (or slice) through torch's dispatcher, with the same base, sizes
// and offset as binding.views gives it, and the interpreter lock is released
// meanwhile, so that a load on another thread starts at once.
#include <Python.h>

#include <ATen/Functions.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "sllm.h"

namespace {

// by SLLM_DTYPE_*
constexpr int64_t kItemSize[] = {4, 2, 2, 1};
constexpr at::ScalarType kType[] = {at::kFloat, at::kHalf, at::kBFloat16, at::kChar};

// `typed` holds the views of buf made so far, one per dtype
at::Tensor view_of(const at::Tensor& buf, at::Tensor* typed, const sllm_tensor_info& t) {
    const int64_t isz = kItemSize[t.dtype], off = (int64_t)t.offset;
    if (buf.storage_offset() % isz || off % isz)  // off its element alignment: raw bytes
        return at::slice(buf, 0, off, off + (int64_t)t.nbytes);
    int64_t strides[SLLM_MAX_NDIM], acc = 1;
    for (uint32_t d = t.ndim; d-- > 0;) {
        strides[d] = acc;
        acc *= std::max<int64_t>(t.shape[d], 1);
    }
    at::Tensor& base = typed[t.dtype];
    if (!base.defined()) base = at::slice(buf, 0, 0, buf.numel() / isz * isz).view(kType[t.dtype]);
    // counted from the start of the storage, not of the typed view
    return at::as_strided(base, at::IntArrayRef(t.shape, t.ndim), at::IntArrayRef(strides, t.ndim),
                          base.storage_offset() + off / isz);
}

// build(buf, table address, n, names_read) -> dict.  The table's names belong to
// the handle: they are copied first, and names_read (a callable or None) is
// called when that is done, after which the handle may be closed.
PyObject* build(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    HANDLE_TH_ERRORS
    if (nargs != 4 || !THPVariable_Check(args[0])) {
        PyErr_SetString(PyExc_TypeError, "build(buf, table, n, names_read)");
        return nullptr;
    }
    const at::Tensor buf = THPVariable_Unpack(args[0]);
    const auto* table = static_cast<const sllm_tensor_info*>(PyLong_AsVoidPtr(args[1]));
    const uint64_t n = PyLong_AsUnsignedLongLong(args[2]);
    if (PyErr_Occurred()) return nullptr;

    std::string names;  // each with its NUL
    at::Tensor typed[4];
    std::vector<at::Tensor> views;
    views.reserve(n);
    bool failed = false;
    {
        pybind11::gil_scoped_release no_gil;
        for (uint64_t i = 0; i < n; ++i) names.append(table[i].name, std::strlen(table[i].name) + 1);
        if (args[3] != Py_None) {
            pybind11::gil_scoped_acquire gil;
            auto r = pybind11::reinterpret_steal<pybind11::object>(PyObject_CallNoArgs(args[3]));
            failed = !r;
        }
        for (uint64_t i = 0; i < n && !failed; ++i) views.push_back(view_of(buf, typed, table[i]));
    }
    if (failed) return nullptr;
    pybind11::object out = pybind11::reinterpret_steal<pybind11::object>(PyDict_New());
    if (!out) return nullptr;
    const char* at = names.c_str();
    for (uint64_t i = 0; i < n; ++i, at += std::strlen(at) + 1) {
        auto name = pybind11::reinterpret_steal<pybind11::object>(PyUnicode_FromString(at));
        if (!name) return nullptr;
        auto v = pybind11::reinterpret_steal<pybind11::object>(THPVariable_Wrap(std::move(views[i])));
        if (!v || PyDict_SetItem(out.ptr(), name.ptr(), v.ptr()) != 0) return nullptr;
    }
    return out.release().ptr();
    END_HANDLE_TH_ERRORS
}

PyMethodDef kMethods[] = {{"build", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(build)), METH_FASTCALL,
                           "build(buf, table, n, names_read) -> {name: view}"},
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_views", "Views over a loaded buffer.", -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// TORCH_VERSION lets the binding refuse a builder made for another torch.
PyMODINIT_FUNC PyInit__views(void) {
    PyObject* m = PyModule_Create(&kModule);
    if (m && PyModule_AddStringConstant(m, "TORCH_VERSION", TORCH_VERSION) != 0) Py_CLEAR(m);
    return m;
}
