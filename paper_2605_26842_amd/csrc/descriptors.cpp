// Fills the descriptor arrays of the C ABI from lists of tensors (host code; nothing of it runs on a GPU).
//
// A step of many small tensors is bound by what stands before its launches, and most of that was reading pointers, shapes and
// dtypes of every tensor through the interpreter: 0.9 us a tensor, 46 us for 49 gains of 4096 and two vectors whose kernel takes 5.
// Read from the tensors themselves it is a few hundredths of a microsecond a tensor.  Only the ordinary case is handled
// here: whatever else a list may hold, the functions return 0 without touching the interpreter's error state, and the caller
// goes through the tensors one by one and says what is wrong.
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mona.h"

namespace {

// the items of a list or tuple, or nothing
PyObject** items(PyObject* list, Py_ssize_t n) {
  if (PyList_CheckExact(list)) return PyList_GET_SIZE(list) == n ? PySequence_Fast_ITEMS(list) : nullptr;
  if (PyTuple_CheckExact(list)) return PyTuple_GET_SIZE(list) == n ? PySequence_Fast_ITEMS(list) : nullptr;
  return nullptr;
}

// a contiguous strided tensor of one of the two dtypes, or nothing
const at::Tensor* plain(PyObject* o, int32_t* dtype) {
  if (!THPVariable_Check(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || t.layout() != at::kStrided || !t.is_contiguous()) return nullptr;
  if (t.scalar_type() == at::kFloat) *dtype = MONA_F32;
  else if (t.scalar_type() == at::kBFloat16) *dtype = MONA_BF16;
  else return nullptr;
  return &t;
}

// calls f(i, parameter, its dtype, gradient, its dtype) for every pair of the two lists while it returns true
template <typename F>
int each_pair(PyObject* params, PyObject* grads, int64_t n, F&& f) {
  try {
    PyObject** const ps = items(params, n);
    PyObject** const gs = items(grads, n);
    if (!ps || !gs) return 0;
    for (int64_t i = 0; i < n; ++i) {
      int32_t wd, gd;
      const at::Tensor* const w = plain(ps[i], &wd);
      const at::Tensor* const g = plain(gs[i], &gd);
      if (!w || !g || w->sizes() != g->sizes() || !f(i, *w, wd, *g, gd)) return 0;
    }
    return 1;
  } catch (...) {
    return 0;
  }
}

}  // namespace

extern "C" {

int mona_fill_vectors(PyObject* params, PyObject* grads, int64_t n, mona_vector* out) {
  return each_pair(params, grads, n, [&](int64_t i, const at::Tensor& w, int32_t wd, const at::Tensor& g, int32_t gd) {
    out[i].w = w.data_ptr();
    out[i].g = g.data_ptr();
    out[i].n = w.numel();
    out[i].w_dtype = wd;
    out[i].g_dtype = gd;
    return true;
  });
}

int mona_fill_matrices(PyObject* params, PyObject* grads, int64_t n, mona_matrix* out) {
  return each_pair(params, grads, n, [&](int64_t i, const at::Tensor& w, int32_t wd, const at::Tensor& g, int32_t gd) {
    if (w.dim() != 2 || w.size(0) > INT32_MAX || w.size(1) > INT32_MAX) return false;
    out[i].w = w.data_ptr();
    out[i].g = g.data_ptr();
    out[i].m = (int32_t)w.size(0);
    out[i].n = (int32_t)w.size(1);
    out[i].w_dtype = wd;
    out[i].g_dtype = gd;
    return true;
  });
}

// the addresses of arrays shaped like the parameters, of dtype `dtype`
int mona_fill_slots(PyObject* params, PyObject* slots, int64_t n, int32_t dtype, void** out) {
  return each_pair(params, slots, n, [&](int64_t i, const at::Tensor&, int32_t, const at::Tensor& s, int32_t sd) {
    out[i] = s.data_ptr();
    return sd == dtype;
  });
}

}  // extern "C"
