// The tensors over a blocks handle's arrays, for the Python binding (module
// _hgviews): the accessors of include/hg.h called and their device arrays
// wrapped as tensors in one native call.  A mini-batch has some tens to hundreds
// of arrays, and through ctypes and __cuda_array_interface__ each took about
// 4 us of the caller's thread (121 us for the 30 arrays of a small mini-batch
// whose own call takes 126).
//
// Every function takes the handle as an integer, the owner (the Blocks object,
// which every returned tensor keeps alive) and the wanted device index (-1:
// where the array is).  A failed accessor's status is returned as an int; the
// accessors are those of the library that the binding has loaded (bind()).
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "hg.h"

namespace {

struct Api {
  decltype(&hg_blocks_nodes) nodes = nullptr;
  decltype(&hg_blocks_edges) edges = nullptr;
  decltype(&hg_blocks_input_nodes) input_nodes = nullptr;
  decltype(&hg_blocks_features) features = nullptr;
  decltype(&hg_blocks_seeds) seeds = nullptr;
  decltype(&hg_blocks_edge_pairs) edge_pairs = nullptr;
} api;

// A new reference, dropped unless it is released.
struct Ref {
  PyObject *o;
  explicit Ref(PyObject *x) : o(x) {}
  Ref(const Ref &) = delete;
  ~Ref() { Py_XDECREF(o); }
  PyObject *release() {
    PyObject *x = o;
    o = nullptr;
    return x;
  }
};

// Drops a reference; any thread may call it.
void drop(void *owner) {
  if (!Py_IsInitialized()) return;  // the interpreter has ended
  const PyGILState_STATE gil = PyGILState_Ensure();
  Py_DECREF(static_cast<PyObject *>(owner));
  PyGILState_Release(gil);
}

// A tensor of this shape over the device memory at p, holding a reference to
// owner; an empty one of its own when there is nothing to show.
PyObject *wrap(const void *p, at::IntArrayRef shape, at::ScalarType type, PyObject *owner,
               int64_t device) {
  int64_t n = 1;
  for (int64_t d : shape) n *= d;
  const auto where = device < 0 ? at::Device(at::kCUDA) : at::Device(at::kCUDA, int8_t(device));
  at::Tensor t;
  if (n == 0 || !p) {
    t = at::empty(shape, at::TensorOptions().dtype(type).device(where));
  } else {
    // (the maker owns the reference from here on: a failed one drops it)
    Py_INCREF(owner);
    t = at::for_blob(const_cast<void *>(p), shape)
            .context(owner, drop)
            .options(at::TensorOptions().dtype(type).device(at::kCUDA))  // the device of p
            .make_tensor();
    if (device >= 0 && t.device() != where) t = t.to(where);
  }
  return THPVariable_Wrap(std::move(t));
}

// The arguments of a call as integers; false with a Python error set.
bool integers(PyObject *const *args, int64_t *out, int n) {
  for (int i = 0; i < n; ++i) {
    out[i] = PyLong_AsLongLong(args[i]);
    if (out[i] == -1 && PyErr_Occurred()) return false;
  }
  return true;
}

// Checks the argument count (integers, then the owner) and reads the integers.
bool arguments(PyObject *const *args, Py_ssize_t n, int ints, int64_t *v) {
  if (n != ints + 1) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return false;
  }
  if (!api.nodes) {
    PyErr_SetString(PyExc_RuntimeError, "bind() has not been called");
    return false;
  }
  return integers(args, v, ints);
}

const hg_blocks *blocks(int64_t h) { return reinterpret_cast<const hg_blocks *>(h); }

// A call's body: C++ exceptions become Python errors.
template <typename F>
PyObject *guarded(F f) {
  try {
    return f();
  } catch (const std::exception &e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// (a, b, ...) from new references, any of which may be NULL (an error).
template <int N>
PyObject *tuple(Ref (&x)[N]) {
  for (const Ref &r : x)
    if (!r.o) return nullptr;
  PyObject *t = PyTuple_New(N);
  for (int i = 0; t && i < N; ++i) PyTuple_SET_ITEM(t, i, x[i].release());
  return t;
}

// nodes(handle, hop, ntype, device, owner) -> (n_dst, src_gid)
PyObject *nodes(PyObject *, PyObject *const *args, Py_ssize_t n) {
  int64_t v[4];
  if (!arguments(args, n, 4, v)) return nullptr;
  return guarded([&]() -> PyObject * {
    int64_t nd = 0, ns = 0;
    const int64_t *p = nullptr;
    const hg_status st = api.nodes(blocks(v[0]), int32_t(v[1]), int32_t(v[2]), &nd, &ns, &p);
    if (st != HG_OK) return PyLong_FromLong(st);
    Ref x[2] = {Ref(PyLong_FromLongLong(nd)),
                Ref(wrap(p, {p ? ns : 0}, at::kLong, args[4], v[3]))};
    return tuple(x);
  });
}

// edges(handle, hop, etype, dst_type, device, owner)
//   -> (indptr, src_local, dst_local, eid)
PyObject *edges(PyObject *, PyObject *const *args, Py_ssize_t n) {
  int64_t v[5];
  if (!arguments(args, n, 5, v)) return nullptr;
  return guarded([&]() -> PyObject * {
    int64_t ne = 0, nd = 0;
    const int64_t *ip = nullptr, *eid = nullptr;
    const int32_t *sl = nullptr, *dl = nullptr;
    hg_status st = api.edges(blocks(v[0]), int32_t(v[1]), int32_t(v[2]), &ne, &ip, &sl, &dl, &eid);
    if (st == HG_OK)
      st = api.nodes(blocks(v[0]), int32_t(v[1]), int32_t(v[3]), &nd, nullptr, nullptr);
    if (st != HG_OK) return PyLong_FromLong(st);
    PyObject *const owner = args[5];
    // (no indptr: an empty array, as for every absent array)
    Ref x[4] = {Ref(wrap(ip, {ip ? nd + 1 : 0}, at::kLong, owner, v[4])),
                Ref(wrap(sl, {sl ? ne : 0}, at::kInt, owner, v[4])),
                Ref(wrap(dl, {dl ? ne : 0}, at::kInt, owner, v[4])),
                Ref(wrap(eid, {eid ? ne : 0}, at::kLong, owner, v[4]))};
    return tuple(x);
  });
}

// input_nodes(handle, ntype, device, owner), seeds(...) -> gid
template <typename Get>
PyObject *gids(PyObject *const *args, Py_ssize_t n, Get get) {
  int64_t v[3];
  if (!arguments(args, n, 3, v)) return nullptr;
  return guarded([&]() -> PyObject * {
    int64_t rows = 0;
    const int64_t *p = nullptr;
    const hg_status st = get()(blocks(v[0]), int32_t(v[1]), &rows, &p);
    if (st != HG_OK) return PyLong_FromLong(st);
    return wrap(p, {p ? rows : 0}, at::kLong, args[3], v[2]);
  });
}
PyObject *input_nodes(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return gids(args, n, [] { return api.input_nodes; });
}
PyObject *seeds(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return gids(args, n, [] { return api.seeds; });
}

// features(handle, ntype, dim, dtype, device, owner) -> [rows, dim] or None;
// dtype: hg_dtype
PyObject *features(PyObject *, PyObject *const *args, Py_ssize_t n) {
  int64_t v[5];
  if (!arguments(args, n, 5, v)) return nullptr;
  return guarded([&]() -> PyObject * {
    int64_t rows = 0;
    const void *p = nullptr;
    const hg_status st = api.features(blocks(v[0]), int32_t(v[1]), &rows, &p);
    if (st != HG_OK) return PyLong_FromLong(st);
    if (!p) Py_RETURN_NONE;
    const at::ScalarType type =
        v[3] == HG_DT_F32 ? at::kFloat : (v[3] == HG_DT_F16 ? at::kHalf : at::kBFloat16);
    return wrap(p, {rows, v[2]}, type, args[5], v[4]);
  });
}

// edge_pairs(handle, etype, device, owner) -> (pos_src, pos_dst, neg_dst)
PyObject *edge_pairs(PyObject *, PyObject *const *args, Py_ssize_t n) {
  int64_t v[3];
  if (!arguments(args, n, 3, v)) return nullptr;
  return guarded([&]() -> PyObject * {
    int64_t np = 0, nn = 0;
    const int32_t *ps = nullptr, *pd = nullptr, *pn = nullptr;
    const hg_status st = api.edge_pairs(blocks(v[0]), int32_t(v[1]), &np, &ps, &pd, &nn, &pn);
    if (st != HG_OK) return PyLong_FromLong(st);
    Ref x[3] = {Ref(wrap(ps, {ps ? np : 0}, at::kInt, args[3], v[2])),
                Ref(wrap(pd, {pd ? np : 0}, at::kInt, args[3], v[2])),
                Ref(wrap(pn, {pn ? nn : 0}, at::kInt, args[3], v[2]))};
    return tuple(x);
  });
}

// bind(nodes, edges, input_nodes, features, seeds, edge_pairs): the addresses
// of the accessors
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n) {
  int64_t v[6];
  if (n != 6) {
    PyErr_SetString(PyExc_TypeError, "bind() takes six addresses");
    return nullptr;
  }
  if (!integers(args, v, 6)) return nullptr;
  api.nodes = reinterpret_cast<decltype(api.nodes)>(v[0]);
  api.edges = reinterpret_cast<decltype(api.edges)>(v[1]);
  api.input_nodes = reinterpret_cast<decltype(api.input_nodes)>(v[2]);
  api.features = reinterpret_cast<decltype(api.features)>(v[3]);
  api.seeds = reinterpret_cast<decltype(api.seeds)>(v[4]);
  api.edge_pairs = reinterpret_cast<decltype(api.edge_pairs)>(v[5]);
  Py_RETURN_NONE;
}

template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyMethodDef method(const char *name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL,
          nullptr};
}

PyMethodDef methods[] = {method<bind>("bind"),
                         method<nodes>("nodes"),
                         method<edges>("edges"),
                         method<input_nodes>("input_nodes"),
                         method<seeds>("seeds"),
                         method<features>("features"),
                         method<edge_pairs>("edge_pairs"),
                         {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_hgviews", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__hgviews(void) { return PyModule_Create(&module); }
