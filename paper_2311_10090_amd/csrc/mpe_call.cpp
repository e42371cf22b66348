// Host path of the Python binding's hot calls (reset, step, rollout, rollout_ac, set_*): argument checks, device
// guard, current stream and the call into libmpe in one native function each.
//
// What bounds it: a single mpe_step is a kernel of a few microseconds, so the time of a call is host work.  Measured
// per step() call of 64 environments: 9.2 us with ctypes and torch's Python accessors (2.9 us of it the lookup of the
// current stream, 1.35 us the device context manager, 1.1 us the pointer checks, the rest ctypes and the launch).
// Here the same checks are a few loads each, and what remains is the launch.
//
// Every function takes (handle, device index, ...) and returns the library's return code; a tensor argument is a
// tensor or None, and must be a contiguous device tensor of the stated type (AssertionError otherwise, as in the
// Python helpers).  The lock of the interpreter is released around the library call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mpe.h"

namespace {

// One call's arguments, read in order; the first failure sets the Python error and `ok` to false.
struct Args {
  PyObject* const* v;
  Py_ssize_t n, at = 0;
  bool ok;

  Args(PyObject* const* args, Py_ssize_t nargs, Py_ssize_t want) : v(args), n(nargs), ok(nargs == want) {
    if (!ok) PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, nargs);
  }
  unsigned long long integer() {
    if (!ok) return 0;
    const unsigned long long x = PyLong_AsUnsignedLongLongMask(v[at++]);
    if (x == static_cast<unsigned long long>(-1) && PyErr_Occurred()) ok = false;
    return x;
  }
  void* pointer(at::ScalarType type) {
    if (!ok) return nullptr;
    PyObject* o = v[at++];
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) {
      PyErr_SetString(PyExc_TypeError, "expected a tensor or None");
      ok = false;
      return nullptr;
    }
    // A tensor without storage (the arguments inside a function transform) throws when it is asked for its address:
    // raised as Python's own accessors raise it, never let through the interpreter's C frames.
    try {
      const at::Tensor& t = THPVariable_Unpack(o);
      if (!t.is_cuda() || !t.is_contiguous()) {
        PyErr_SetString(PyExc_AssertionError, "device-resident contiguous tensor required");
      } else if (t.scalar_type() != type) {
        PyErr_Format(PyExc_AssertionError, "expected %s, got %s", c10::toString(type), c10::toString(t.scalar_type()));
      } else {
        return t.data_ptr();
      }
    } catch (...) {
      torch::translate_exception_to_python(std::current_exception());
    }
    ok = false;
    return nullptr;
  }
  float* f32() { return static_cast<float*>(pointer(at::kFloat)); }
  uint8_t* u8() { return static_cast<uint8_t*>(pointer(at::kByte)); }
};

// Runs `call(stream)` with the handle's device current and its current stream.
template <typename F>
PyObject* run(const Args& a, int device, F call) {
  if (!a.ok) return nullptr;
  int rc;
  try {
    const c10::DeviceGuard guard(c10::Device(c10::DeviceType::CUDA, c10::DeviceIndex(device)));
    void* stream = c10::hip::getCurrentHIPStream(c10::DeviceIndex(device)).stream();
    Py_BEGIN_ALLOW_THREADS
    rc = call(stream);
    Py_END_ALLOW_THREADS
  } catch (...) {
    torch::translate_exception_to_python(std::current_exception());
    return nullptr;
  }
  // the library's message belongs to this thread: the caller fetches it through mpe_last_error
  return PyLong_FromLong(rc);
}

mpe_env* handle(Args& a) { return reinterpret_cast<mpe_env*>(a.integer()); }

PyObject* py_reset(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 4);
  mpe_env* e = handle(a);
  const int dev = int(a.integer());
  const uint32_t seed = uint32_t(a.integer());
  float* obs = a.f32();
  return run(a, dev, [=](void* s) { return mpe_reset(e, seed, obs, s); });
}

PyObject* py_step(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 6);
  mpe_env* e = handle(a);
  const int dev = int(a.integer());
  const uint8_t* actions = a.u8();
  float* obs = a.f32();
  float* reward = a.f32();
  uint8_t* done = a.u8();
  return run(a, dev, [=](void* s) { return mpe_step(e, actions, obs, reward, done, s); });
}

PyObject* py_rollout(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 8);
  mpe_env* e = handle(a);
  const int dev = int(a.integer());
  const int32_t T = int32_t(a.integer());
  float* obs = a.f32();
  uint8_t* act = a.u8();
  float* rew = a.f32();
  uint8_t* done = a.u8();
  float* last = a.f32();
  return run(a, dev, [=](void* s) { return mpe_rollout(e, T, obs, act, rew, done, last, s); });
}

PyObject* py_rollout_ac(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 11);
  mpe_env* e = handle(a);
  const int dev = int(a.integer());
  const int32_t T = int32_t(a.integer());
  float* obs = a.f32();
  uint8_t* act = a.u8();
  float* logp = a.f32();
  float* value = a.f32();
  float* rew = a.f32();
  uint8_t* done = a.u8();
  float* last = a.f32();
  float* last_value = a.f32();
  return run(a, dev, [=](void* s) { return mpe_rollout_ac(e, T, obs, act, logp, value, rew, done, last, last_value, s); });
}

// set_policy, set_critic, set_gru_policy, set_gru_critic: K weight arrays.
template <typename Fn, int K>
PyObject* set_weights(Fn fn, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 2 + K);
  mpe_env* e = handle(a);
  const int dev = int(a.integer());
  const float* w[K];
  for (int k = 0; k < K; ++k) w[k] = a.f32();
  return run(a, dev, [&](void* s) {
    if constexpr (K == 10) return fn(e, w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7], w[8], w[9], s);
    else if constexpr (K == 6) return fn(e, w[0], w[1], w[2], w[3], w[4], w[5], s);
    else return fn(e, w[0], w[1], w[2], w[3], s);
  });
}
PyObject* py_set_policy(PyObject*, PyObject* const* v, Py_ssize_t n) { return set_weights<decltype(&mpe_set_policy), 6>(&mpe_set_policy, v, n); }
PyObject* py_set_critic(PyObject*, PyObject* const* v, Py_ssize_t n) { return set_weights<decltype(&mpe_set_critic), 6>(&mpe_set_critic, v, n); }
PyObject* py_set_gru_policy(PyObject*, PyObject* const* v, Py_ssize_t n) { return set_weights<decltype(&mpe_set_gru_policy), 10>(&mpe_set_gru_policy, v, n); }
PyObject* py_set_gru_critic(PyObject*, PyObject* const* v, Py_ssize_t n) { return set_weights<decltype(&mpe_set_gru_critic), 4>(&mpe_set_gru_critic, v, n); }

#define MPE_METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&py_##NAME)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MPE_METHOD(reset), MPE_METHOD(step), MPE_METHOD(rollout), MPE_METHOD(rollout_ac), MPE_METHOD(set_policy),
                         MPE_METHOD(set_critic), MPE_METHOD(set_gru_policy), MPE_METHOD(set_gru_critic), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mpe_call", "Native host path of the libmpe binding.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__mpe_call(void) { return PyModule_Create(&module); }
