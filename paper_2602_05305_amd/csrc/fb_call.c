// Native form of the binding's calls (paper_2602_05305_amd/flashblock.py): takes the Python arguments of an entry point, makes the
// C arguments of it and calls it.  Nothing else: which entry points there are, their arguments and what a status means stay with the
// Python module.  Arguments that are not of the plain kinds below, or missing, or of an unknown name, go to the Python function that a
// call stands for (its __wrapped__), which takes or refuses them as it always has.
//
// A reuse step is one kernel of some 3.3 us and its launch costs the host 2.3 us, so the marshalling around it shows: 1.4 us through
// ctypes and Python functions, 0.5 us here.
//
// Every parameter of the entry points is a pointer or an integer, which the x86-64 calling convention passes alike in 64-bit slots.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#define MAX_ARGS 20                          // C arguments of an entry point

// One entry point.  Its i-th C argument (two for a W) is made of Python argument order[i] as kinds[i] says:
//   S, K  shape, paged cache (ctypes structures): the address   P  tensor (or None): its device address
//   W  workspace tensor (or None): address and size in bytes, two C arguments
//   I  integer                                  H  stream: None (the current one), an object with cuda_stream, or a handle
typedef struct {
  PyObject_HEAD
  vectorcallfunc vectorcall;
  PyObject *name, *names, *defaults;         // defaults: of the last arguments
  PyObject *resolve, *stream, *check;        // name -> address; () -> current stream's handle; (status, name) raises
  PyObject *shape, *paged;                   // types of S and K
  PyObject *dict, *weakrefs;                 // attributes (functools.update_wrapper)
  char kinds[MAX_ARGS + 1];
  int order[MAX_ARGS];
  Py_ssize_t n;
  void* fn;
} Call;

static PyObject *g_device, *g_raw_stream;    // () -> current device, (device) -> its current stream's handle; or unset
static PyObject *s_data_ptr, *s_numel, *s_element_size, *s_cuda_stream, *s_wrapped;

typedef int64_t A;
typedef int (*F)(A, A, A, A, A, A, A, A, A, A, A, A, A, A, A, A, A, A, A, A);

static int as_int(PyObject* o, A* out) {
  if (!PyLong_Check(o)) {
    PyErr_Format(PyExc_TypeError, "an integer is expected, not %s", Py_TYPE(o)->tp_name);
    return -1;
  }
  *out = (A)PyLong_AsUnsignedLongLongMask(o);
  return *out == -1 && PyErr_Occurred() ? -1 : 0;
}

static int from_method(PyObject* o, PyObject* method, A* out) {
  PyObject* r = PyObject_CallMethodNoArgs(o, method);
  if (!r) return -1;
  const int e = as_int(r, out);
  Py_DECREF(r);
  return e;
}

static int marshal(Call* c, PyObject* const* args, A* a) {
  int n = 0;
  for (Py_ssize_t i = 0; i < c->n; ++i) {
    PyObject* o = args[c->order[i]];
    switch (c->kinds[i]) {
      case 'S':
      case 'K': {
        PyObject* type = c->kinds[i] == 'S' ? c->shape : c->paged;
        if (!PyObject_TypeCheck(o, (PyTypeObject*)type)) {
          PyErr_Format(PyExc_TypeError, "%U: %s instead of %s", c->name, Py_TYPE(o)->tp_name, ((PyTypeObject*)type)->tp_name);
          return -1;
        }
        Py_buffer b;
        if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) < 0) return -1;
        a[n++] = (A)(intptr_t)b.buf;
        PyBuffer_Release(&b);                // the caller's argument keeps it in place
        break;
      }
      case 'P':
        if (o == Py_None) a[n++] = 0;
        else if (from_method(o, s_data_ptr, &a[n++]) < 0) return -1;
        break;
      case 'W':
        if (o == Py_None) {
          if (c->order[i] < c->n - PyTuple_GET_SIZE(c->defaults)) {
            PyErr_Format(PyExc_AttributeError, "%U: no workspace", c->name);
            return -1;
          }
          a[n++] = 0;
          a[n++] = 0;
        } else {
          A count, size;
          if (from_method(o, s_data_ptr, &a[n++]) < 0 || from_method(o, s_numel, &count) < 0 || from_method(o, s_element_size, &size) < 0) return -1;
          a[n++] = count * size;
        }
        break;
      case 'I':
        if (as_int(o, &a[n++]) < 0) return -1;
        break;
      default: {                             // H
        PyObject* r;
        if (PyLong_Check(o)) {
          Py_INCREF(o);
          r = o;
        } else if (o != Py_None) {
          r = PyObject_GetAttr(o, s_cuda_stream);
        } else if (g_device) {
          PyObject* d = PyObject_CallNoArgs(g_device);
          r = d ? PyObject_CallOneArg(g_raw_stream, d) : NULL;
          Py_XDECREF(d);
        } else {
          r = PyObject_CallNoArgs(c->stream);
        }
        if (!r) return -1;
        const int e = as_int(r, &a[n++]);
        Py_DECREF(r);
        if (e < 0) return -1;
      }
    }
  }
  return n;
}

// Arguments by name and the defaults, into all[]; 0 with or without an exception: not a call of this function.
static int bind(Call* c, PyObject* const* args, Py_ssize_t given, PyObject* kw, PyObject** all) {
  const Py_ssize_t nkw = kw ? PyTuple_GET_SIZE(kw) : 0, nd = PyTuple_GET_SIZE(c->defaults);
  for (Py_ssize_t i = 0; i < c->n; ++i) all[i] = i < given ? args[i] : NULL;
  for (Py_ssize_t k = 0; k < nkw; ++k) {
    PyObject* key = PyTuple_GET_ITEM(kw, k);
    Py_ssize_t i = 0;
    for (; i < c->n; ++i) {
      PyObject* name = PyTuple_GET_ITEM(c->names, i);
      if (name == key || PyUnicode_Compare(name, key) == 0) break;
    }
    if (i == c->n || all[i]) return 0;
    all[i] = args[given + k];
  }
  for (Py_ssize_t i = 0; i < c->n; ++i)
    if (!all[i]) {
      if (i < c->n - nd) return 0;
      all[i] = PyTuple_GET_ITEM(c->defaults, i - (c->n - nd));
    }
  return 1;
}

// The same call by the Python function.
static PyObject* by_python(Call* c, PyObject* const* args, size_t nargsf, PyObject* kw) {
  PyObject* fn = c->dict ? PyDict_GetItemWithError(c->dict, s_wrapped) : NULL;
  if (!fn) return PyErr_Occurred() ? NULL : PyErr_Format(PyExc_TypeError, "%U: arguments that are not of the native call's kinds", c->name);
  PyErr_Clear();
  Py_INCREF(fn);
  PyObject* r = PyObject_Vectorcall(fn, args, nargsf & ~PY_VECTORCALL_ARGUMENTS_OFFSET, kw);
  Py_DECREF(fn);
  return r;
}

static PyObject* call(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kw) {
  Call* c = (Call*)self;
  const Py_ssize_t given = PyVectorcall_NARGS(nargsf);
  PyObject* all[MAX_ARGS];
  PyObject* const* bound = args;
  if (given != c->n || (kw && PyTuple_GET_SIZE(kw))) {
    if (given > c->n || !bind(c, args, given, kw, all)) return by_python(c, args, nargsf, kw);
    bound = all;
  }
  if (!c->fn) {                              // the first call: the library is loaded now
    PyObject* r = PyObject_CallOneArg(c->resolve, c->name);
    if (!r) return NULL;
    void* fn = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    if (!fn) return PyErr_Occurred() ? NULL : PyErr_Format(PyExc_RuntimeError, "%U: no address", c->name);
    c->fn = fn;
  }
  A a[MAX_ARGS] = {0};
  if (marshal(c, bound, a) < 0) {
    if (!PyErr_ExceptionMatches(PyExc_TypeError) && !PyErr_ExceptionMatches(PyExc_AttributeError)) return NULL;
    return by_python(c, args, nargsf, kw);
  }
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = ((F)c->fn)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12], a[13], a[14], a[15], a[16], a[17], a[18], a[19]);
  Py_END_ALLOW_THREADS
  if (status) {
    PyObject* r = PyObject_CallFunction(c->check, "iO", status, c->name);
    if (!r) return NULL;
    Py_DECREF(r);
  }
  Py_RETURN_NONE;
}

// Pickled and copied as a function is: by its name in its module.
static PyObject* call_reduce(PyObject* self, PyObject* unused) {
  PyObject* name = ((Call*)self)->name;
  Py_INCREF(name);
  return name;
}

// On a class, a method, as a function is.
static PyObject* call_get(PyObject* self, PyObject* of, PyObject* type) {
  if (!of || of == Py_None) {
    Py_INCREF(self);
    return self;
  }
  return PyMethod_New(self, of);
}

static void call_dealloc(PyObject* self) {
  Call* c = (Call*)self;
  if (c->weakrefs) PyObject_ClearWeakRefs(self);
  Py_XDECREF(c->dict);
  Py_XDECREF(c->name); Py_XDECREF(c->names); Py_XDECREF(c->defaults);
  Py_XDECREF(c->resolve); Py_XDECREF(c->stream); Py_XDECREF(c->check); Py_XDECREF(c->shape); Py_XDECREF(c->paged);
  Py_TYPE(self)->tp_free(self);
}

static PyObject* call_repr(PyObject* self) { return PyUnicode_FromFormat("<native call %U>", ((Call*)self)->name); }

// Call(name, names, defaults, kinds, order, resolve, stream, check, shape type, paged cache type)
static PyObject* call_new(PyTypeObject* type, PyObject* args, PyObject* kw) {
  PyObject *name, *names, *defaults, *order, *resolve, *stream, *check, *shape, *paged;
  const char* kinds;
  if (kw && PyDict_GET_SIZE(kw)) return PyErr_Format(PyExc_TypeError, "Call: positional arguments only");
  if (!PyArg_ParseTuple(args, "UO!O!sO!OOOO!O!", &name, &PyTuple_Type, &names, &PyTuple_Type, &defaults, &kinds, &PyTuple_Type, &order,
                        &resolve, &stream, &check, &PyType_Type, &shape, &PyType_Type, &paged)) return NULL;
  const Py_ssize_t n = PyTuple_GET_SIZE(names);
  Py_ssize_t slots = 0;
  for (const char* k = kinds; *k; ++k) {
    if (!strchr("SKPWIH", *k)) return PyErr_Format(PyExc_ValueError, "Call: unknown kind in '%s'", kinds);
    slots += *k == 'W' ? 2 : 1;
  }
  if ((Py_ssize_t)strlen(kinds) != n || PyTuple_GET_SIZE(order) != n || slots > MAX_ARGS || PyTuple_GET_SIZE(defaults) > n)
    return PyErr_Format(PyExc_ValueError, "Call: arguments of %U", name);
  Call* c = (Call*)type->tp_alloc(type, 0);
  if (!c) return NULL;
  c->vectorcall = call;
  Py_INCREF(name); Py_INCREF(names); Py_INCREF(defaults); Py_INCREF(resolve); Py_INCREF(stream); Py_INCREF(check); Py_INCREF(shape); Py_INCREF(paged);
  c->name = name; c->names = names; c->defaults = defaults; c->resolve = resolve; c->stream = stream; c->check = check;
  c->shape = shape; c->paged = paged;
  strcpy(c->kinds, kinds);
  c->n = n;
  c->fn = NULL;
  for (Py_ssize_t i = 0; i < n; ++i) {
    const long at = PyLong_AsLong(PyTuple_GET_ITEM(order, i));
    if (at < 0 || at >= n) {
      Py_DECREF(c);
      return PyErr_Occurred() ? NULL : PyErr_Format(PyExc_ValueError, "Call: order of %U", name);
    }
    c->order[i] = (int)at;
  }
  return (PyObject*)c;
}

static PyObject* set_stream_getters(PyObject* self, PyObject* args) {
  PyObject *device, *stream;
  if (!PyArg_ParseTuple(args, "OO", &device, &stream)) return NULL;
  Py_INCREF(device);
  Py_INCREF(stream);
  Py_XSETREF(g_raw_stream, stream);
  Py_XSETREF(g_device, device);
  Py_RETURN_NONE;
}

static PyMethodDef methods[] = {{"set_stream_getters", set_stream_getters, METH_VARARGS, NULL}, {NULL}};

static PyMethodDef call_methods[] = {{"__reduce__", call_reduce, METH_NOARGS, NULL}, {NULL}};

static PyGetSetDef call_getset[] = {{"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, NULL, NULL}, {NULL}};

static PyTypeObject CallType = {
    PyVarObject_HEAD_INIT(NULL, 0).tp_name = "paper_2602_05305_amd._fbcall.Call",
    .tp_basicsize = sizeof(Call),
    .tp_dealloc = call_dealloc,
    .tp_repr = call_repr,
    .tp_call = PyVectorcall_Call,
    .tp_vectorcall_offset = offsetof(Call, vectorcall),
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_methods = call_methods,
    .tp_getset = call_getset,
    .tp_dictoffset = offsetof(Call, dict),
    .tp_weaklistoffset = offsetof(Call, weakrefs),
    .tp_descr_get = call_get,
    .tp_new = call_new,
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fbcall", NULL, -1, methods};

PyMODINIT_FUNC PyInit__fbcall(void) {
  if (PyType_Ready(&CallType) < 0) return NULL;
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_numel = PyUnicode_InternFromString("numel");
  s_element_size = PyUnicode_InternFromString("element_size");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  s_wrapped = PyUnicode_InternFromString("__wrapped__");
  if (!s_wrapped || !s_data_ptr || !s_numel || !s_element_size || !s_cuda_stream) return NULL;
  PyObject* m = PyModule_Create(&module);
  if (!m) return NULL;
  Py_INCREF(&CallType);
  if (PyModule_AddObject(m, "Call", (PyObject*)&CallType) < 0) return NULL;
  return m;
}
