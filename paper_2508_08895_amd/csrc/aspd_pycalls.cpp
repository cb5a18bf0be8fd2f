// The per-step calls of the Python binding: argument marshalling only, as compiled code.
//
// What bounds the smallest steps is the host.  An append and an attention call take some forty addresses and sizes out of
// the caller's objects; in Python (three ctypes structures and a ctypes call each) that was 17 us a layer where the
// launches themselves take five and the kernels of one short sequence twelve.  Here an address is an attribute and a
// field of the tensor behind it: an append and an attention call 17 -> 1.5 us of host work, a step of one layer in fp32
// 43.6 -> 27.5 us, of four layers over one sequence of 2 300 tokens 107 -> 69, over 27 mixed sequences 113 -> 90 (the kernels
// are what is left).  Nothing is kept from one call for the next: the objects are read anew each time, so
// whatever a program assigns to them counts.
//
// The plain case only: an object of the binding's own class, whose fields are plain tensors, None and ints that fit.
// Everything else goes through the object's struct() method, which defines what is accepted and what is raised.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/device_lazy_init.h>

#include <climits>
#include <cstring>

#include "aspd.h"

namespace {

PyObject *g_kv_type, *g_state_type, *g_step_type;  // the binding's classes (set once, by init)

// The library's entry points, from the binding's own handle of it (set with them): this module is linked against no library,
// so that the calls here and those by ctypes are always calls of one.
#define ASPD_CALLS(X)                                                                                                  \
  X(attn_parallel_decode) X(attn_branch_chunk) X(attn_serial_decode) X(attn_full_sequence)                             \
  X(attn_parallel_decode_static) X(rope_append) X(build_branch_meta) X(sequence_plan_bytes) X(build_sequence_meta)
#define ASPD_POINTER(name) decltype(&aspd_##name) name;
struct {
  ASPD_CALLS(ASPD_POINTER)
} g_lib;
#undef ASPD_POINTER

// Names, interned at import.
#define ASPD_NAMES(X)                                                                                                  \
  X(k) X(v) X(block_tables) X(num_q_heads) X(B) X(NB) X(stage_base) X(seq_len) X(cu_branches) X(branch_len)            \
  X(slot_owner) X(owner_stride) X(fault) X(main_pos) X(stage_open) X(NQ) X(max_new_per_seq) X(max_workgroups)          \
  X(shared_mask) X(cu_new) X(cu_seq_new) X(q_seq) X(q_branch) X(position_ids) X(logical_slot) X(slot_mapping)          \
  X(kv_len) X(plan) X(plan_key) X(pos_mode) X(data_ptr) X(numel) X(element_size) X(cuda_stream)
#define ASPD_DECLARE(name) PyObject* n_##name;
ASPD_NAMES(ASPD_DECLARE)
PyObject* n_struct;
#undef ASPD_DECLARE

// A new reference, given back at the end of the scope.
struct Ref {
  PyObject* o;
  explicit Ref(PyObject* o_) : o(o_) {}
  ~Ref() { Py_XDECREF(o); }
  Ref(const Ref&) = delete;
  Ref& operator=(const Ref&) = delete;
};

inline bool plain_tensor(PyObject* o) { return THPVariable_CheckExact(o); }

// Fields of an object of the plain case; `ok` turns false at the first that is not plain (never with an exception set).
struct Fields {
  PyObject* obj;
  bool ok = true;
  explicit Fields(PyObject* o) : obj(o) {}

  // The object holds the attribute for as long as the GIL is held: a borrowed pointer would do but for attributes made
  // on access, hence a reference.
  PyObject* get(PyObject* name) {
    PyObject* v = PyObject_GetAttr(obj, name);
    if (!v) {
      PyErr_Clear();  // (struct() raises it again)
      ok = false;
    }
    return v;
  }
  template <typename T>
  void ptr(PyObject* name, T** out) {
    Ref v(get(name));
    if (!v.o) return;
    if (v.o == Py_None) *out = nullptr;
    else if (plain_tensor(v.o)) *out = (T*)THPVariable_Unpack(v.o).data_ptr();
    else ok = false;
  }
  void i32(PyObject* name, int32_t* out) {
    Ref v(get(name));
    if (!v.o) return;
    if (!PyLong_CheckExact(v.o)) {
      ok = false;
      return;
    }
    int over = 0;
    const long x = PyLong_AsLongAndOverflow(v.o, &over);
    if (over || x < INT32_MIN || x > INT32_MAX) ok = false;
    else *out = (int32_t)x;
  }
};

// The general case: obj.struct(), a ctypes structure of the same layout.
template <typename S>
bool from_struct(PyObject* obj, S* out) {
  Ref s(PyObject_CallMethodObjArgs(obj, n_struct, nullptr));
  if (!s.o) return false;
  Py_buffer view;
  if (PyObject_GetBuffer(s.o, &view, PyBUF_SIMPLE) != 0) return false;
  const bool fits = view.len == (Py_ssize_t)sizeof(S);
  if (fits) memcpy(out, view.buf, sizeof(S));
  PyBuffer_Release(&view);
  if (!fits) PyErr_Format(PyExc_TypeError, "struct() of a %s has another size", Py_TYPE(obj)->tp_name);
  return fits;
}

bool fill(PyObject* obj, aspd_kv* out) {
  if ((PyObject*)Py_TYPE(obj) != g_kv_type) return from_struct(obj, out);
  Fields f(obj);
  Ref k(f.get(n_k)), v(f.get(n_v)), t(f.get(n_block_tables));
  if (!f.ok || !plain_tensor(k.o) || !plain_tensor(v.o) || !plain_tensor(t.o)) return from_struct(obj, out);
  const at::Tensor& kt = THPVariable_Unpack(k.o);
  const at::Tensor& tt = THPVariable_Unpack(t.o);
  if (kt.dim() != 4 || tt.dim() < 2) return from_struct(obj, out);
  const int64_t sizes[5] = {kt.size(0), kt.size(1), kt.size(2), kt.size(3), tt.size(1)};
  for (const int64_t n : sizes)
    if (n > INT32_MAX) return from_struct(obj, out);
  memset(out, 0, sizeof(*out));
  if (kt.scalar_type() == at::kBFloat16) out->dtype = ASPD_BF16;
  else if (kt.scalar_type() == at::kFloat) out->dtype = ASPD_F32;
  else return from_struct(obj, out);
  out->k_cache_d = kt.data_ptr();
  out->v_cache_d = THPVariable_Unpack(v.o).data_ptr();
  out->block_tables_d = (const int32_t*)tt.data_ptr();
  out->num_blocks = (int32_t)sizes[0];
  out->num_kv_heads = (int32_t)sizes[1];
  out->block_size = (int32_t)sizes[2];
  out->head_dim = (int32_t)sizes[3];
  out->max_blocks_per_seq = (int32_t)sizes[4];
  f.i32(n_num_q_heads, &out->num_q_heads);
  return f.ok || from_struct(obj, out);
}

bool fill(PyObject* obj, aspd_state* out) {
  if ((PyObject*)Py_TYPE(obj) != g_state_type) return from_struct(obj, out);
  memset(out, 0, sizeof(*out));
  Fields f(obj);
  f.i32(n_B, &out->B);
  f.i32(n_NB, &out->NB);
  f.ptr(n_stage_base, &out->stage_base_d);
  f.ptr(n_seq_len, &out->seq_len_d);
  f.ptr(n_cu_branches, &out->cu_branches_d);
  f.ptr(n_branch_len, &out->branch_len_d);
  f.ptr(n_slot_owner, &out->slot_owner_d);
  f.i32(n_owner_stride, &out->owner_stride);
  f.ptr(n_fault, &out->fault_d);
  f.ptr(n_main_pos, &out->main_pos_d);
  f.ptr(n_stage_open, &out->stage_open_d);
  return f.ok || from_struct(obj, out);
}

bool fill(PyObject* obj, aspd_step* out) {
  if ((PyObject*)Py_TYPE(obj) != g_step_type) return from_struct(obj, out);
  memset(out, 0, sizeof(*out));
  Fields f(obj);
  f.i32(n_NQ, &out->NQ);
  f.i32(n_max_new_per_seq, &out->max_new_per_seq);
  f.i32(n_max_workgroups, &out->max_workgroups);
  f.i32(n_shared_mask, &out->shared_mask);
  f.ptr(n_cu_new, &out->cu_new_d);
  f.ptr(n_cu_seq_new, &out->cu_seq_new_d);
  f.ptr(n_q_seq, &out->q_seq_d);
  f.ptr(n_q_branch, &out->q_branch_d);
  f.ptr(n_position_ids, &out->position_ids_d);
  f.ptr(n_logical_slot, &out->logical_slot_d);
  f.ptr(n_slot_mapping, &out->slot_mapping_d);
  f.ptr(n_kv_len, &out->kv_len_d);
  Ref plan(f.get(n_plan)), key(f.get(n_plan_key));
  if (f.ok && plain_tensor(plan.o)) {
    const at::Tensor& t = THPVariable_Unpack(plan.o);
    out->plan_d = (int32_t*)t.data_ptr();
    out->plan_bytes = (size_t)t.numel() * t.element_size();
  } else if (plan.o != Py_None) {
    f.ok = false;
  }
  if (f.ok && PyLong_CheckExact(key.o)) out->plan_key = PyLong_AsUnsignedLongLongMask(key.o);
  else f.ok = false;
  return f.ok || from_struct(obj, out);
}

// The address of a tensor (None: null), or of anything else that has data_ptr().
bool address(PyObject* o, void** out) {
  if (plain_tensor(o)) {
    *out = THPVariable_Unpack(o).data_ptr();
    return true;
  }
  if (o == Py_None) {
    *out = nullptr;
    return true;
  }
  Ref p(PyObject_CallMethodObjArgs(o, n_data_ptr, nullptr));
  if (!p.o) return false;
  if (p.o == Py_None) {
    *out = nullptr;
    return true;
  }
  if (!PyLong_Check(p.o)) {
    PyErr_Format(PyExc_TypeError, "data_ptr() of a %s is no int", Py_TYPE(o)->tp_name);
    return false;
  }
  *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(p.o);
  return !PyErr_Occurred();
}

bool bytes_of(PyObject* o, size_t* out) {
  *out = 0;
  if (o == Py_None) return true;
  if (plain_tensor(o)) {
    const at::Tensor& t = THPVariable_Unpack(o);
    *out = (size_t)t.numel() * t.element_size();
    return true;
  }
  Ref n(PyObject_CallMethodObjArgs(o, n_numel, nullptr));
  if (!n.o) return false;
  Ref e(PyObject_CallMethodObjArgs(o, n_element_size, nullptr));
  if (!e.o) return false;
  Ref x(PyNumber_Multiply(n.o, e.o));
  if (!x.o) return false;
  *out = (size_t)PyLong_AsUnsignedLongLongMask(x.o);
  return !PyErr_Occurred();
}

bool int_of(PyObject* o, int32_t* out) {  // as a ctypes int32 argument takes it: whatever stands for a whole number
  Ref i(PyNumber_Index(o));
  if (!i.o) return false;
  *out = (int32_t)PyLong_AsUnsignedLongMask(i.o);
  return !PyErr_Occurred();
}

bool float_of(PyObject* o, float* out) {
  const double d = PyFloat_AsDouble(o);
  *out = (float)d;
  return !(d == -1.0 && PyErr_Occurred());
}

// None: the stream that is current on the current device.
bool stream_of(PyObject* o, void** out) {
  if (o == Py_None) {
    torch::utils::device_lazy_init(at::kCUDA);  // (raises where there is no device)
    *out = (void*)c10::hip::getCurrentHIPStream().stream();
    return true;
  }
  Ref s(PyObject_GetAttr(o, n_cuda_stream));
  if (!s.o) return false;
  if (s.o == Py_None) {
    *out = nullptr;
    return true;
  }
  if (!PyLong_Check(s.o)) {
    PyErr_SetString(PyExc_TypeError, "cuda_stream is no int");
    return false;
  }
  *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(s.o);
  return !PyErr_Occurred();
}

// Every call: with the exceptions of torch turned into Python's, and a count of arguments that the binding's own
// wrappers always give.
template <typename Body>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, Body body) {
  if (n != want) {
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
    return nullptr;
  }
  try {
    return body();
  } catch (python_error& e) {
    e.restore();
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}

enum { PARALLEL, CHUNK, SERIAL, SEQUENCE, STATIC_PARALLEL };

// (which, kv, state, step, q, out, lse, sm_scale, workspace, stream) -> status
PyObject* py_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&]() -> PyObject* {
    int32_t which;
    aspd_kv kv;
    aspd_state st;
    aspd_step sp;
    void *q, *out, *lse, *ws, *stream;
    size_t ws_bytes;
    float scale;
    if (!int_of(a[0], &which) || !fill(a[1], &kv) || !fill(a[2], &st) || !fill(a[3], &sp) || !bytes_of(a[8], &ws_bytes) ||
        !address(a[4], &q) || !address(a[5], &out) || !address(a[6], &lse) || !float_of(a[7], &scale) ||
        !address(a[8], &ws) || !stream_of(a[9], &stream))
      return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    switch (which) {
      case PARALLEL: rc = g_lib.attn_parallel_decode(&kv, &st, &sp, q, out, (float*)lse, scale, ws, ws_bytes, stream); break;
      case CHUNK: rc = g_lib.attn_branch_chunk(&kv, &st, &sp, q, out, (float*)lse, scale, ws, ws_bytes, stream); break;
      case SERIAL: rc = g_lib.attn_serial_decode(&kv, &st, &sp, q, out, (float*)lse, scale, ws, ws_bytes, stream); break;
      case SEQUENCE: rc = g_lib.attn_full_sequence(&kv, &st, &sp, q, out, (float*)lse, scale, ws, ws_bytes, stream); break;
      default: rc = g_lib.attn_parallel_decode_static(&kv, &st, &sp, q, out, (float*)lse, scale, stream); break;
    }
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(rc);
  });
}

// (kv, step, q, k_new, v_new, rope_theta, stream) -> status
PyObject* py_rope_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 7, [&]() -> PyObject* {
    aspd_kv kv;
    aspd_step sp;
    void *q, *k, *v, *stream;
    float theta;
    if (!fill(a[0], &kv) || !fill(a[1], &sp) || !address(a[2], &q) || !address(a[3], &k) || !address(a[4], &v) ||
        !float_of(a[5], &theta) || !stream_of(a[6], &stream))
      return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = g_lib.rope_append(&kv, &sp, q, k, v, theta, stream);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(rc);
  });
}

// (kv, state, stage, new_len, step or None, stream) -> status; sets step.plan_key, the one host field the library writes
PyObject* py_build_branch_meta(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 6, [&]() -> PyObject* {
    aspd_kv kv;
    aspd_state st;
    aspd_step sp;
    int32_t stage, pos_mode;
    void *new_len, *stream;
    const bool with_step = a[4] != Py_None;
    if (!fill(a[0], &kv) || !fill(a[1], &st) || (with_step && !fill(a[4], &sp))) return nullptr;
    Ref mode(PyObject_GetAttr(a[1], n_pos_mode));
    if (!mode.o || !int_of(a[2], &stage) || !int_of(mode.o, &pos_mode) || !address(a[3], &new_len) ||
        !stream_of(a[5], &stream))
      return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = g_lib.build_branch_meta(&kv, &st, stage, pos_mode, (const int32_t*)new_len, with_step ? &sp : nullptr, stream);
    Py_END_ALLOW_THREADS;
    if (rc == ASPD_OK && with_step) {
      Ref key(PyLong_FromUnsignedLongLong(sp.plan_key));
      if (!key.o || PyObject_SetAttr(a[4], n_plan_key, key.o) != 0) return nullptr;
    }
    return PyLong_FromLong(rc);
  });
}

// (kv, B, NQ) -> bytes
PyObject* py_sequence_plan_bytes(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 3, [&]() -> PyObject* {
    aspd_kv kv;
    int32_t B, NQ;
    if (!fill(a[0], &kv) || !int_of(a[1], &B) || !int_of(a[2], &NQ)) return nullptr;
    return PyLong_FromSize_t(g_lib.sequence_plan_bytes(&kv, B, NQ));
  });
}

// (kv, state, runs, cu_runs, run_branch, run_len, step, stream) -> status; sets step.plan_key
PyObject* py_build_sequence_meta(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 8, [&]() -> PyObject* {
    aspd_kv kv;
    aspd_state st;
    aspd_step sp;
    aspd_layout lay;
    int32_t pos_mode;
    void *cu_runs, *run_branch, *run_len, *stream;
    if (!fill(a[0], &kv) || !fill(a[1], &st) || !fill(a[6], &sp) || !int_of(a[2], &lay.num_runs) || !address(a[3], &cu_runs) ||
        !address(a[4], &run_branch) || !address(a[5], &run_len))
      return nullptr;
    Ref mode(PyObject_GetAttr(a[1], n_pos_mode));
    if (!mode.o || !int_of(mode.o, &pos_mode) || !stream_of(a[7], &stream)) return nullptr;
    lay.cu_runs_d = (const int32_t*)cu_runs;
    lay.run_branch_d = (const int32_t*)run_branch;
    lay.run_len_d = (const int32_t*)run_len;
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = g_lib.build_sequence_meta(&kv, &st, &lay, pos_mode, &sp, stream);
    Py_END_ALLOW_THREADS;
    if (rc == ASPD_OK) {
      Ref key(PyLong_FromUnsignedLongLong(sp.plan_key));
      if (!key.o || PyObject_SetAttr(a[6], n_plan_key, key.o) != 0) return nullptr;
    }
    return PyLong_FromLong(rc);
  });
}

// (kv, state, step) -> their structures as bytes, as the calls above see them
PyObject* py_structs(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 3, [&]() -> PyObject* {
    aspd_kv kv;
    aspd_state st;
    aspd_step sp;
    if (!fill(a[0], &kv) || !fill(a[1], &st) || !fill(a[2], &sp)) return nullptr;
    return Py_BuildValue("(y#y#y#)", (const char*)&kv, (Py_ssize_t)sizeof(kv), (const char*)&st, (Py_ssize_t)sizeof(st),
                         (const char*)&sp, (Py_ssize_t)sizeof(sp));
  });
}

// (KVCache, BatchState, Step, {name: address}): the classes of the plain case and the library's entry points
PyObject* py_init(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 4, [&]() -> PyObject* {
    auto lib = g_lib;
#define ASPD_LOOK_UP(name)                                                                                             \
  {                                                                                                                    \
    Ref address(PyMapping_GetItemString(a[3], "aspd_" #name));                                                         \
    if (!address.o) return nullptr;                                                                                    \
    lib.name = (decltype(lib.name))PyLong_AsVoidPtr(address.o);                                                        \
    if (PyErr_Occurred()) return nullptr;                                                                              \
  }
    ASPD_CALLS(ASPD_LOOK_UP)
#undef ASPD_LOOK_UP
    g_lib = lib;
    PyObject** const to[3] = {&g_kv_type, &g_state_type, &g_step_type};
    for (int i = 0; i < 3; ++i) {
      Py_INCREF(a[i]);
      Py_XSETREF(*to[i], a[i]);
    }
    Py_RETURN_NONE;
  });
}

#define ASPD_METHOD(name) {#name, (PyCFunction)(void (*)())py_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ASPD_METHOD(attn), ASPD_METHOD(rope_append), ASPD_METHOD(build_branch_meta),
                         ASPD_METHOD(sequence_plan_bytes), ASPD_METHOD(build_sequence_meta), ASPD_METHOD(structs),
                         ASPD_METHOD(init), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_pycalls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycalls() {
#define ASPD_INTERN(name) \
  if (!(n_##name = PyUnicode_InternFromString(#name))) return nullptr;
  ASPD_NAMES(ASPD_INTERN)
  ASPD_INTERN(struct)
#undef ASPD_INTERN
  return PyModule_Create(&module_def);
}
