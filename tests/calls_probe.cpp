// The way of a call through csrc/calls.cpp with entry points of the test's own: probe(what) calls one that throws, or that takes its time,
// rows_later(graph) one that looks at the graph after half a second.
#include "calls.cpp"

#include <chrono>
#include <stdexcept>
#include <thread>

namespace {

HGNN_CALL(probe, 1) {
  const int what = r.integer(a[0]);
  return [=]() -> hgnn_status {
    if (what == 1) throw std::bad_alloc();
    if (what == 2) throw std::runtime_error("out of luck");
    if (what == 3) std::this_thread::sleep_for(std::chrono::milliseconds(500));
    return hgnn_status(what == 4 ? HGNN_EINVAL : HGNN_OK);
  };
} HGNN_END

HGNN_CALL(rows_later, 1) {
  const hgnn_csr g = r.graph(a[0]);
  return [=] {
    std::this_thread::sleep_for(std::chrono::milliseconds(500));
    return hgnn_status(g.nrows);
  };
} HGNN_END

PyMethodDef probe_methods[] = {HGNN_METHOD(probe), HGNN_METHOD(rows_later), {nullptr, nullptr, 0, nullptr}};
PyModuleDef probe_module = {PyModuleDef_HEAD_INIT, "calls_probe", nullptr, -1, probe_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_calls_probe() {
  PyInit__calls();  // attribute names
  g_raw_stream = Py_NewRef(Py_None);
  return PyModule_Create(&probe_module);
}
