// Suggestion dicts -> bbo_mlp_hparams records, as a CPython extension: a call with thousands of suggestions otherwise
// spends as long on this conversion as the GPU on the models.
//
// pack(suggestions, address): fills the records at `address` (room for all) from the front and returns how many
// it did.  It stops in front of the first suggestion that is not a plain dict of plain values (int, float, bool, str, a
// list or tuple of ints): the caller converts that one in Python, where its types say what the numbers are.
// 2048 suggestions: 1.8 ms in Python, 0.25 ms here.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/bbo_mlp.h"

enum { HIDDEN, SOLVER, NESTEROV, BATCH, EPOCHS, LR, ALPHA, MOMENTUM, BETA1, BETA2, EPS, SEED, POWER_T, TOL, PATIENCE, VAL, N_KEYS };
static const char* const NAMES[N_KEYS] = {"hidden", "solver", "nesterov", "batch_size", "epochs", "lr", "alpha", "momentum",
                                          "beta1", "beta2", "eps", "seed", "power_t", "tol", "n_iter_no_change",
                                          "validation_fraction"};
static PyObject* keys[N_KEYS];

// Each returns 1 if it has set *out, 0 if the value is not plain.
static inline int get_int(PyObject* v, int32_t* out) {
  if (!PyLong_CheckExact(v) && !PyBool_Check(v)) return 0;
  *out = (int32_t)PyLong_AsUnsignedLongMask(v);  // as ctypes takes it
  return 1;
}
static inline int get_float(PyObject* v, float* out) {
  if (PyFloat_CheckExact(v)) return *out = (float)PyFloat_AS_DOUBLE(v), 1;
  if (!PyLong_CheckExact(v)) return 0;
  const double x = PyLong_AsDouble(v);
  if (x == -1.0 && PyErr_Occurred()) return PyErr_Clear(), 0;
  *out = (float)x;
  return 1;
}
static int get_hidden(PyObject* v, bbo_mlp_hparams* h) {
  if (!PyList_CheckExact(v) && !PyTuple_CheckExact(v)) return 0;
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(v);
  for (Py_ssize_t i = 0; i < n && i < BBO_MAX_HIDDEN; i++) {
    PyObject* w = PySequence_Fast_GET_ITEM(v, i);
    if (!PyLong_CheckExact(w)) return 0;
    h->hidden[i] = (int32_t)PyLong_AsUnsignedLongMask(w);
  }
  h->n_hidden = (int32_t)n;
  return 1;
}
// The entries of the dict in its own order: keys written in a program are interned, so that a key is known by its
// address (and is most often the one after the last).
static int pack_one(PyObject* d, bbo_mlp_hparams* h) {
  static const bbo_mlp_hparams defaults = {.solver = BBO_ADAM, .epochs = 1, .lr = 1e-3f, .momentum = 0.9f, .beta1 = 0.9f,
                                           .beta2 = 0.999f, .eps = 1e-8f};
  if (!PyDict_CheckExact(d)) return 0;
  *h = defaults;
  PyObject *key, *v;
  Py_ssize_t pos = 0;
  int k = 0, ok = 1;
  while (ok && PyDict_Next(d, &pos, &key, &v)) {
    int tries = 0;
    while (keys[k] != key && tries < N_KEYS) {
      k = k + 1 < N_KEYS ? k + 1 : 0;
      tries++;
    }
    if (keys[k] != key) {  // some other key, or one of ours built at run time
      if (!PyUnicode_CheckExact(key) || !PyUnicode_CHECK_INTERNED(key)) return 0;
      continue;
    }
    switch (k) {
      case HIDDEN: ok = get_hidden(v, h); break;
      case SOLVER:
        ok = PyUnicode_CheckExact(v);
        if (ok) h->solver = PyUnicode_CompareWithASCIIString(v, "sgd") == 0 ? BBO_SGD : BBO_ADAM;
        break;
      case NESTEROV:
        ok = PyBool_Check(v);
        h->nesterov = v == Py_True;
        break;
      case BATCH: ok = get_int(v, &h->batch_size); break;
      case EPOCHS: ok = get_int(v, &h->epochs); break;
      case LR: ok = get_float(v, &h->lr); break;
      case ALPHA: ok = get_float(v, &h->alpha); break;
      case MOMENTUM: ok = get_float(v, &h->momentum); break;
      case BETA1: ok = get_float(v, &h->beta1); break;
      case BETA2: ok = get_float(v, &h->beta2); break;
      case EPS: ok = get_float(v, &h->eps); break;
      case SEED:
        ok = PyLong_CheckExact(v);
        if (ok) h->seed = PyLong_AsUnsignedLongLongMask(v);
        break;
      case POWER_T: ok = get_float(v, &h->power_t); break;
      case TOL: ok = get_float(v, &h->tol); break;
      case PATIENCE: ok = get_int(v, &h->n_iter_no_change); break;
      case VAL: ok = get_float(v, &h->validation_fraction); break;
    }
  }
  return ok;
}

static PyObject* pack(PyObject* self, PyObject* args) {
  PyObject* list;
  unsigned long long address;
  Py_ssize_t first = 0, i;
  (void)self;
  if (!PyArg_ParseTuple(args, "OK|n", &list, &address, &first)) return NULL;
  if (!PyList_CheckExact(list) && !PyTuple_CheckExact(list)) return PyLong_FromSsize_t(first);
  bbo_mlp_hparams* h = (bbo_mlp_hparams*)(uintptr_t)address;
  for (i = first; i < PySequence_Fast_GET_SIZE(list); i++)
    if (!pack_one(PySequence_Fast_GET_ITEM(list, i), h + i)) break;
  if (PyErr_Occurred()) return NULL;
  return PyLong_FromSsize_t(i);
}

static PyMethodDef methods[] = {{"pack", pack, METH_VARARGS, "pack(suggestions, address, first=0) -> suggestions done"},
                                {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pack", NULL, -1, methods, NULL, NULL, NULL, NULL};
PyMODINIT_FUNC PyInit__pack(void) {
  for (int k = 0; k < N_KEYS; k++) {
    keys[k] = PyUnicode_InternFromString(NAMES[k]);
    if (!keys[k]) return NULL;
  }
  return PyModule_Create(&module);
}
