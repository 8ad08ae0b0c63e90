// Python calls of libeagletv.so without ctypes.  A step makes dozens of calls whose kernels take 3 ... 15 us each, and
// marshalling a dozen tensors through Python (three attribute calls per tensor, a stream object, ctypes conversions) took
// 9 us per attention call: longer than the kernel.  Here one template turns the arguments into those of the C prototype in
// eagletv.h: a pointer parameter takes a device-resident contiguous tensor or None, a descriptor any object with the buffer
// of that struct, an integer an int or what has __index__ (numpy's integers, tensors of one); the trailing stream is the
// current one.  The GIL is released around the call.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <type_traits>
#include <utility>

#include "eagletv.h"

namespace {

struct Refused {};  // a Python exception is set

template <class T>
constexpr bool is_desc = std::is_same_v<T, const etv_attn_desc *> || std::is_same_v<T, const etv_commit_desc *> ||
                         std::is_same_v<T, const etv_cache_desc *>;

template <class T>
T arg(PyObject *o) {
    if constexpr (std::is_integral_v<T>) {
        if (!PyIndex_Check(o)) {
            PyErr_Format(PyExc_TypeError, "int expected instead of %s", Py_TYPE(o)->tp_name);
            throw Refused{};
        }
        const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);  // takes ints and what has __index__
        if (v == ~0ull && PyErr_Occurred()) throw Refused{};
        return static_cast<T>(v);
    } else if constexpr (is_desc<T>) {
        // the caller's reference keeps the object, and with it the memory of a ctypes structure, for the whole call
        Py_buffer view;
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Refused{};
        const bool fits = view.len >= (Py_ssize_t)sizeof(std::remove_pointer_t<T>);
        T p = static_cast<T>(view.buf);
        PyBuffer_Release(&view);
        if (!fits) {
            PyErr_SetString(PyExc_ValueError, "descriptor too small");
            throw Refused{};
        }
        return p;
    } else {
        static_assert(std::is_pointer_v<T>);
        if (o == Py_None) return nullptr;
        if (!THPVariable_Check(o)) {
            PyErr_Format(PyExc_TypeError, "tensor expected instead of %s", Py_TYPE(o)->tp_name);
            throw Refused{};
        }
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous()) {
            PyErr_SetString(PyExc_AssertionError, "device-resident contiguous tensors only");
            throw Refused{};
        }
        return static_cast<T>(t.data_ptr());
    }
}

template <class... A, std::size_t... I>
int32_t apply(int32_t (*f)(A...), PyObject *const *args, std::index_sequence<I...>) {
    std::tuple<A...> v;
    ((std::get<I>(v) = arg<std::tuple_element_t<I, std::tuple<A...>>>(args[I])), ...);  // left to right; the stream is last
    std::get<sizeof...(A) - 1>(v) = c10::hip::getCurrentHIPStream().stream();
    int32_t rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = std::apply(f, v);
    Py_END_ALLOW_THREADS;
    return rc;
}

template <class... A>
constexpr Py_ssize_t arity(int32_t (*)(A...)) { return sizeof...(A) - 1; }

template <auto F>
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    constexpr Py_ssize_t want = arity(F);
    if (n != want) return PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, n);
    try {
        return PyLong_FromLong(apply(F, args, std::make_index_sequence<want>{}));
    } catch (const Refused &) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// empty_i32(like, sizes...): an int32 tensor on the device of `like`
PyObject *empty_i32(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n < 1 || n > 5 || !THPVariable_Check(args[0])) return PyErr_Format(PyExc_TypeError, "empty_i32(tensor, sizes...)");
    int64_t sizes[4];
    for (Py_ssize_t i = 1; i < n; i++) {
        sizes[i - 1] = PyLong_AsLongLong(args[i]);
        if (sizes[i - 1] == -1 && PyErr_Occurred()) return nullptr;
    }
    const at::TensorOptions o = at::TensorOptions().dtype(at::kInt).device(THPVariable_Unpack(args[0]).device());
    return THPVariable_Wrap(at::empty(at::IntArrayRef(sizes, n - 1), o));
    END_HANDLE_TH_ERRORS
}

// commit_desc(kt, k_cache, block_table or None, W): the descriptor's bytes, from the shapes; None where they are not those of a step's tree
// rows and caches (kt None among them), which the Python caller then names
PyObject *commit_desc(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 4) return PyErr_Format(PyExc_TypeError, "4 arguments expected, got %zd", n);
    const bool paged = args[2] != Py_None;
    if (!THPVariable_Check(args[0]) || !THPVariable_Check(args[1]) || (paged && !THPVariable_Check(args[2])) || !PyLong_Check(args[3])) Py_RETURN_NONE;
    const at::Tensor &kt = THPVariable_Unpack(args[0]), &cache = THPVariable_Unpack(args[1]);
    if (kt.dim() != 5 || cache.dim() != 5 || kt.size(0) != cache.size(0)) Py_RETURN_NONE;
    etv_commit_desc d{};
    const auto i32 = [](int64_t v) { return static_cast<int32_t>(v); };
    d.n_layers = i32(kt.size(0));
    d.B = i32(kt.size(1));
    d.T_max = i32(kt.size(2));
    d.Hkv = i32(kt.size(3));
    d.d = i32(kt.size(4));
    d.elem_bytes = i32(cache.element_size());
    d.W = static_cast<int32_t>(PyLong_AsUnsignedLongLongMask(args[3]));
    if (paged) {
        const at::Tensor &table = THPVariable_Unpack(args[2]);
        if (table.dim() < 2) Py_RETURN_NONE;
        d.block_size = i32(cache.size(3));
        d.max_blocks = i32(table.size(1));
        d.num_blocks = i32(cache.size(1));
    } else {
        d.P_cap = i32(cache.size(2));
    }
    d.cache_layer_stride = d.n_layers > 1 ? cache.stride(0) : cache.numel();
    return PyBytes_FromStringAndSize(reinterpret_cast<const char *>(&d), sizeof d);
    END_HANDLE_TH_ERRORS
}

#define ETV_METHOD(name) {#name, (PyCFunction)(void (*)(void))call<&etv_##name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ETV_METHOD(build_tree_mask), ETV_METHOD(tensorize_tree), ETV_METHOD(tree_verify_attention),
                         ETV_METHOD(tree_verify_attention_static), ETV_METHOD(safe_gather_paths), ETV_METHOD(evaluate_posterior),
                         ETV_METHOD(commit_accepted_kv), ETV_METHOD(verify_epilogue), ETV_METHOD(lm_head_argmax),
                         ETV_METHOD(pack_lm_head), ETV_METHOD(replicate_branches), ETV_METHOD(commit_path_indices),
                         {"commit_desc", (PyCFunction)(void (*)(void))commit_desc, METH_FASTCALL, nullptr},
                         {"empty_i32", (PyCFunction)(void (*)(void))empty_i32, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
