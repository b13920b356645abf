// The two calls that a decoding loop makes, codegemm_gemm and codegemm_gemm_grouped, as functions of a Python extension module.  Through ctypes
// such a call spends 2.8 us in the interpreter and in argument conversion before it reaches the library, of the 8 us that
// an eager call of a small layer takes in all (its kernels take 3); here 0.6.  Only the plain form of a call is handled: positional
// arguments, Desc and Plan themselves, tensors (anything with data_ptr()), integer addresses or None.  Every other form, and every
// argument that the plain form refuses, goes to the ctypes functions, which then do and raise what they always did.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstddef>
#include <cstdint>
#include <initializer_list>

#include "codegemm.h"

namespace {

typedef int (*gemm_t)(const codegemm_desc*, const codegemm_plan*, const void*, const uint8_t*, const void*, const void*, void*, void*, size_t, void*);
typedef int (*grouped_t)(const codegemm_desc*, const codegemm_plan*, const void*, const codegemm_group_member*, int32_t, void*, size_t, void*);

// Set by prepare() when the binding is imported and by use() when it has loaded a library; with the GIL held, as they are read.
PyTypeObject* desc_type = nullptr;
PyTypeObject* plan_type = nullptr;
PyObject *slow_gemm = nullptr, *slow_grouped = nullptr, *check = nullptr, *data_ptr = nullptr;
gemm_t gemm_at = nullptr;
grouped_t grouped_at = nullptr;
constexpr Py_ssize_t kMaxMembers = 4;

// The bytes of a ctypes structure, held while the view lives.
struct View {
    Py_buffer b;
    bool held = false;
    bool of(PyObject* o, size_t bytes)
    {
        held = PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) == 0;
        return held && (size_t)b.len == bytes;
    }
    ~View() { if (held) PyBuffer_Release(&b); }
};

enum Form { kPlain, kOther, kRaised };

// Address of a tensor, an integer or None.  What a data_ptr() raises is the caller's to see, but for AttributeError, which sends the
// ctypes forms on to int(o).
Form address(PyObject* o, void** at)
{
    if (o == Py_None) { *at = nullptr; return kPlain; }
    if (PyLong_CheckExact(o)) *at = PyLong_AsVoidPtr(o);
    else {
        PyObject* n = PyObject_CallMethodNoArgs(o, data_ptr);
        if (!n) return PyErr_ExceptionMatches(PyExc_AttributeError) ? kOther : kRaised;
        if (!PyLong_CheckExact(n)) { Py_DECREF(n); return kOther; }
        *at = PyLong_AsVoidPtr(n);
        Py_DECREF(n);
    }
    return *at != nullptr || !PyErr_Occurred() ? kPlain : kOther;
}

bool size(PyObject* o, size_t* n)
{
    if (!PyLong_CheckExact(o)) return false;
    *n = PyLong_AsSize_t(o);
    return !(*n == (size_t)-1 && PyErr_Occurred());
}

bool structures(PyObject* d, PyObject* p, View* desc, View* plan)
{
    return Py_TYPE(d) == desc_type && desc->of(d, sizeof(codegemm_desc)) &&
           (p == Py_None || (Py_TYPE(p) == plan_type && plan->of(p, sizeof(codegemm_plan))));
}

PyObject* slowly(PyObject* how, PyObject* const* args, Py_ssize_t nargs, PyObject* names)
{
    if (!how) { PyErr_SetString(PyExc_RuntimeError, "prepare() has not been called"); return nullptr; }
    PyErr_Clear();                                     // whatever stood in the way of the plain form: it will be met again
    return PyObject_Vectorcall(how, args, (size_t)nargs, names);
}

PyObject* result(int status, const char* where)
{
    if (status != 0) return PyObject_CallFunction(check, "is", status, where);
    Py_RETURN_NONE;
}

// (desc, plan, x, packed_codes, codebooks, scales, y, workspace, workspace_bytes, stream=0)
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n, PyObject* names)
{
    View desc, plan;
    void *at[6], *stream = nullptr;
    size_t bytes;
    Form form = gemm_at && !names && (n == 9 || n == 10) && structures(a[0], a[1], &desc, &plan) ? kPlain : kOther;
    for (int k = 0; form == kPlain && k < 6; ++k) form = address(a[2 + k], &at[k]);
    if (form == kRaised) return nullptr;
    if (form == kOther || !size(a[8], &bytes) || (n == 10 && !(PyLong_CheckExact(a[9]) && address(a[9], &stream) == kPlain))) return slowly(slow_gemm, a, n, names);
    const gemm_t call = gemm_at;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call(static_cast<const codegemm_desc*>(desc.b.buf), plan.held ? static_cast<const codegemm_plan*>(plan.b.buf) : nullptr, at[0],
                  static_cast<const uint8_t*>(at[1]), at[2], at[3], at[4], at[5], bytes, stream);
    Py_END_ALLOW_THREADS
    return result(status, "codegemm_gemm");
}

// (desc, plan, x, members, workspace, workspace_bytes, stream=0); members: (out_features, packed_codes, codebooks, scales, y) each
PyObject* gemm_grouped(PyObject*, PyObject* const* a, Py_ssize_t n, PyObject* names)
{
    View desc, plan;
    void *x, *workspace, *stream = nullptr;
    size_t bytes;
    codegemm_group_member group[kMaxMembers] = {};
    int32_t count = 0;
    Form form = grouped_at && !names && (n == 6 || n == 7) && structures(a[0], a[1], &desc, &plan) &&
                (PyList_CheckExact(a[3]) || PyTuple_CheckExact(a[3])) && PySequence_Fast_GET_SIZE(a[3]) <= kMaxMembers ? kPlain : kOther;
    // (a data_ptr() may run any Python, so the list is asked for its length again, and members are held while they are read)
    for (; form == kPlain && count < PySequence_Fast_GET_SIZE(a[3]) && count < kMaxMembers; ++count) {
        PyObject* m = PySequence_Fast_GET_ITEM(a[3], count);
        Py_INCREF(m);
        form = kOther;
        if (PyTuple_CheckExact(m) && PyTuple_GET_SIZE(m) == 5 && PyLong_CheckExact(PyTuple_GET_ITEM(m, 0))) {
            const long rows = PyLong_AsLong(PyTuple_GET_ITEM(m, 0));
            void* at[4];
            if (rows >= INT32_MIN && rows <= INT32_MAX && !(rows == -1 && PyErr_Occurred())) form = kPlain;
            for (int k = 0; form == kPlain && k < 4; ++k) form = address(PyTuple_GET_ITEM(m, 1 + k), &at[k]);
            if (form == kPlain) {
                group[count].out_features = (int32_t)rows;
                group[count].packed_codes = static_cast<const uint8_t*>(at[0]);
                group[count].codebooks = at[1];
                group[count].scales = at[2];
                group[count].y = at[3];
            }
        }
        Py_DECREF(m);
    }
    if (form == kPlain) form = address(a[2], &x);
    if (form == kPlain) form = address(a[4], &workspace);
    if (form == kRaised) return nullptr;
    if (form == kOther || !size(a[5], &bytes) || (n == 7 && !(PyLong_CheckExact(a[6]) && address(a[6], &stream) == kPlain)))
        return slowly(slow_grouped, a, n, names);
    const grouped_t call = grouped_at;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call(static_cast<const codegemm_desc*>(desc.b.buf), plan.held ? static_cast<const codegemm_plan*>(plan.b.buf) : nullptr, x, group, count,
                  workspace, bytes, stream);
    Py_END_ALLOW_THREADS
    return result(status, "codegemm_gemm_grouped");
}

// (Desc, Plan, the ctypes forms of the two calls, what raises for a status)
PyObject* prepare(PyObject*, PyObject* args)
{
    PyObject *d, *p, *one, *group, *raise;
    if (!PyArg_ParseTuple(args, "O!O!OOO", &PyType_Type, &d, &PyType_Type, &p, &one, &group, &raise)) return nullptr;
    for (PyObject* o : {d, p, one, group, raise}) Py_INCREF(o);        // for the life of the process
    desc_type = reinterpret_cast<PyTypeObject*>(d);
    plan_type = reinterpret_cast<PyTypeObject*>(p);
    slow_gemm = one;
    slow_grouped = group;
    check = raise;
    Py_RETURN_NONE;
}

// (address of codegemm_gemm, address of codegemm_gemm_grouped)
PyObject* use(PyObject*, PyObject* args)
{
    unsigned long long one, group;
    if (!PyArg_ParseTuple(args, "KK", &one, &group)) return nullptr;
    gemm_at = reinterpret_cast<gemm_t>(static_cast<uintptr_t>(one));
    grouped_at = reinterpret_cast<grouped_t>(static_cast<uintptr_t>(group));
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"codegemm_gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(gemm)), METH_FASTCALL | METH_KEYWORDS,
     "codegemm_gemm(desc, plan, x, packed_codes, codebooks, scales, y, workspace, workspace_bytes, stream=0)\n--\n\n"},
    {"codegemm_gemm_grouped", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(gemm_grouped)), METH_FASTCALL | METH_KEYWORDS,
     "codegemm_gemm_grouped(desc, plan, x, members, workspace, workspace_bytes, stream=0)\n--\n\n"
     "members: sequence of (out_features, packed_codes, codebooks, scales, y), tensors or raw device addresses."},
    {"prepare", prepare, METH_VARARGS, nullptr},
    {"use", use, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void)
{
    data_ptr = PyUnicode_InternFromString("data_ptr");
    return data_ptr ? PyModule_Create(&module) : nullptr;
}
