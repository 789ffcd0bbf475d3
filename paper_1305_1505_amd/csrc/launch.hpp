// Kernel launches, eager or recorded into a HIP graph.
//
// A thread that holds a GraphRecorder records: its launches become kernel nodes of that graph, each
// after the one before.  Nothing is captured from a stream, because while any stream of the process
// is being captured the runtime refuses hipMemcpy to every thread (hipErrorStreamCaptureImplicit) and
// the refused call spoils the capture: a server that captured as it ran would fail its clients' copies.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace pin {

class GraphRecorder {
 public:
  GraphRecorder();
  ~GraphRecorder();
  GraphRecorder(const GraphRecorder&) = delete;
  GraphRecorder& operator=(const GraphRecorder&) = delete;

  // the calling thread's recorder, or null
  static GraphRecorder* current();
  void add(const void* kernel, dim3 grid, dim3 block, void** args);
  hipGraphExec_t instantiate();

 private:
  hipGraph_t graph_ = nullptr;
  hipGraphNode_t last_ = nullptr;
};

template <typename... P>
void launch(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t s, std::common_type_t<P>... args) {
  if (GraphRecorder* r = GraphRecorder::current()) {
    void* p[] = {const_cast<void*>(static_cast<const void*>(&args))...};
    r->add(reinterpret_cast<const void*>(kernel), grid, block, p);
  } else {
    hipLaunchKernelGGL(kernel, grid, block, 0, s, args...);
  }
}

}  // namespace pin
