// Native argument marshalling for the Python binding: call(index, address, args)
// checks the tensors of one libdora entry point (plain tensors, on the GPU,
// contiguous, the required type) and calls it at that address, without the
// GIL.  Anything else -- another object, a tensor subclass, an
// active torch function mode, an argument that fails a check -- returns
// NotImplemented, and the binding marshals the call through ctypes, which
// raises the errors.  ctypes and the checks in Python cost about 5 us of a
// call's 9; this costs about 0.3 us.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "dora.h"

namespace {

union Arg {
  void* p;
  int64_t n;
  float f;
};

// Argument kinds: F, I, L, A are float32, int32, int64 and any-type tensors
// (lower case: or None), n an integer, e a float, s an address.
struct Entry {
  const char* kinds;
  int (*call)(void* fn, const Arg* a);
};

template <class T>
T* ptr(const Arg& a) {
  return static_cast<T*>(a.p);
}
// The entry point of the declared function's type at address fn (the loaded library's).
template <class F>
F* at_address(F&, void* fn) {
  return reinterpret_cast<F*>(fn);
}
int32_t i32(const Arg& a) { return static_cast<int32_t>(a.n); }
dora_dtype type_of(const Arg& a) { return static_cast<dora_dtype>(a.n); }

// The order is that of _ENTRIES in the binding.
const Entry kEntries[] = {
    {"FIAinnnnnIIAnIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_select_pack, fn)(ptr<float>(a[0]), ptr<int32_t>(a[1]), a[2].p, ptr<int32_t>(a[3]), a[4].n, i32(a[5]),
                               i32(a[6]), i32(a[7]), type_of(a[8]), ptr<int32_t>(a[9]), ptr<int32_t>(a[10]), a[11].p,
                               a[12].n, ptr<int32_t>(a[13]), a[14].p);
     }},
    {"FIAinnnnnIIAnnnnAnIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_select_pack_plan, fn)(ptr<float>(a[0]), ptr<int32_t>(a[1]), a[2].p, ptr<int32_t>(a[3]), a[4].n,
                                    i32(a[5]), i32(a[6]), i32(a[7]), type_of(a[8]), ptr<int32_t>(a[9]),
                                    ptr<int32_t>(a[10]), a[11].p, a[12].n, i32(a[13]), i32(a[14]), a[15].n, a[16].p,
                                    static_cast<size_t>(a[17].n), ptr<int32_t>(a[18]), a[19].p);
     }},
    {"FIAAinnnnnIIAnIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_select_pack_residual, fn)(ptr<float>(a[0]), ptr<int32_t>(a[1]), a[2].p, a[3].p, ptr<int32_t>(a[4]),
                                        a[5].n, i32(a[6]), i32(a[7]), i32(a[8]), type_of(a[9]), ptr<int32_t>(a[10]),
                                        ptr<int32_t>(a[11]), a[12].p, a[13].n, ptr<int32_t>(a[14]), a[15].p);
     }},
    {"FinnnIIIIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_actor_gate, fn)(ptr<float>(a[0]), ptr<int32_t>(a[1]), i32(a[2]), i32(a[3]), i32(a[4]),
                              ptr<int32_t>(a[5]), ptr<int32_t>(a[6]), ptr<int32_t>(a[7]), ptr<int32_t>(a[8]), a[9].p);
     }},
    {"fnnfinnnIIfIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_actor_decode, fn)(ptr<float>(a[0]), a[1].n, i32(a[2]), ptr<float>(a[3]), ptr<int32_t>(a[4]), a[5].n,
                                i32(a[6]), i32(a[7]), ptr<int32_t>(a[8]), ptr<int32_t>(a[9]), ptr<float>(a[10]),
                                ptr<int32_t>(a[11]), a[12].p);
     }},
    {"FFIinnnIIFnIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_pl_sample, fn)(ptr<float>(a[0]), ptr<float>(a[1]), ptr<int32_t>(a[2]), ptr<int32_t>(a[3]), a[4].n,
                             i32(a[5]), i32(a[6]), ptr<int32_t>(a[7]), ptr<int32_t>(a[8]), ptr<float>(a[9]), a[10].n,
                             ptr<int32_t>(a[11]), a[12].p);
     }},
    {"FIIinnnFIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_pl_logprob, fn)(ptr<float>(a[0]), ptr<int32_t>(a[1]), ptr<int32_t>(a[2]), ptr<int32_t>(a[3]), a[4].n,
                              i32(a[5]), i32(a[6]), ptr<float>(a[7]), ptr<int32_t>(a[8]), a[9].p);
     }},
    {"AInnnnFFeFanIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_lc1_readout, fn)(a[0].p, ptr<int32_t>(a[1]), a[2].n, i32(a[3]), i32(a[4]), type_of(a[5]),
                               ptr<float>(a[6]), ptr<float>(a[7]), a[8].f, ptr<float>(a[9]), a[10].p,
                               static_cast<size_t>(a[11].n), ptr<int32_t>(a[12]), a[13].p);
     }},
    {"InsLLIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_trajectory_flops, fn)(ptr<int32_t>(a[0]), i32(a[1]), ptr<dora_flops_config>(a[2]), ptr<int64_t>(a[3]),
                                    ptr<int64_t>(a[4]), ptr<int32_t>(a[5]), a[6].p);
     }},
    {"InnnnAnIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_varlen_attn_plan, fn)(ptr<int32_t>(a[0]), i32(a[1]), i32(a[2]), i32(a[3]), a[4].n, a[5].p,
                                    static_cast<size_t>(a[6].n), ptr<int32_t>(a[7]), a[8].p);
     }},
    {"AAAInnnnnenAAnIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_varlen_attn_execute, fn)(a[0].p, a[1].p, a[2].p, ptr<int32_t>(a[3]), i32(a[4]), i32(a[5]), i32(a[6]),
                                       i32(a[7]), a[8].n, a[9].f, type_of(a[10]), a[11].p, a[12].p,
                                       static_cast<size_t>(a[13].n), ptr<int32_t>(a[14]), a[15].p);
     }},
    {"AAAInnnnnenAAnIs",
     [](void* fn, const Arg* a) {
       return at_address(dora_varlen_attn, fn)(a[0].p, a[1].p, a[2].p, ptr<int32_t>(a[3]), i32(a[4]), i32(a[5]), i32(a[6]), i32(a[7]),
                               a[8].n, a[9].f, type_of(a[10]), a[11].p, a[12].p, static_cast<size_t>(a[13].n),
                               ptr<int32_t>(a[14]), a[15].p);
     }},
};
constexpr int kMaxArgs = 20;

bool tensor_arg(PyObject* o, char kind, Arg* out) {
  if (o == Py_None) {
    out->p = nullptr;
    return kind >= 'a' && kind <= 'z';
  }
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || !t.is_contiguous()) return false;
  const at::ScalarType want = kind == 'F' || kind == 'f' ? at::kFloat : kind == 'I' || kind == 'i' ? at::kInt : at::kLong;
  if (kind != 'A' && kind != 'a' && t.scalar_type() != want) return false;
  out->p = t.data_ptr();  // throws for tensors without storage
  return true;
}

PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  const long which = nargs > 1 ? PyLong_AsLong(args[0]) : -1;
  void* const fn = nargs > 1 ? PyLong_AsVoidPtr(args[1]) : nullptr;
  if (fn == nullptr || which < 0 || which >= static_cast<long>(sizeof(kEntries) / sizeof(kEntries[0]))) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no such entry point");
    return nullptr;
  }
  const Entry& entry = kEntries[which];
  if (nargs - 2 != static_cast<Py_ssize_t>(strlen(entry.kinds)) || at::impl::torch_function_mode_enabled())
    Py_RETURN_NOTIMPLEMENTED;
  Arg a[kMaxArgs];
  try {
    for (Py_ssize_t i = 0; i + 2 < nargs; ++i) {
      PyObject* o = args[i + 2];
      const char kind = entry.kinds[i];
      if (kind == 'n' || kind == 's') {
        if (!PyLong_CheckExact(o)) Py_RETURN_NOTIMPLEMENTED;
        int overflow = 0;
        a[i].n = PyLong_AsLongLongAndOverflow(o, &overflow);
        if (overflow) Py_RETURN_NOTIMPLEMENTED;
      } else if (kind == 'e') {
        if (!PyFloat_CheckExact(o)) Py_RETURN_NOTIMPLEMENTED;
        a[i].f = static_cast<float>(PyFloat_AS_DOUBLE(o));
      } else if (!tensor_arg(o, kind, &a[i])) {
        Py_RETURN_NOTIMPLEMENTED;
      }
    }
  } catch (...) {
    Py_RETURN_NOTIMPLEMENTED;
  }
  // A launch can wait for room in its queue: let other threads run, as ctypes
  // does.  What an entry point throws is caught where the GIL is not held, and
  // the call is not made again.
  int rc = 0;
  bool threw = false;
  Py_BEGIN_ALLOW_THREADS
  try {
    rc = entry.call(fn, a);
  } catch (...) {
    threw = true;
  }
  Py_END_ALLOW_THREADS
  if (threw) {
    PyErr_SetString(PyExc_RuntimeError, "the entry point threw a C++ exception");
    return nullptr;
  }
  return PyLong_FromLong(rc);
}

PyMethodDef kMethods[] = {
    {"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call)), METH_FASTCALL,
     "call(index, address, *args): the status, or NotImplemented"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_host_call", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host_call() { return PyModule_Create(&kModule); }
