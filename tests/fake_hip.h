// A stand-in for the HIP runtime on the CPU -- TEST INFRASTRUCTURE ONLY.
// Streams are queues that one thread works off in order; an operation may wait
// for a gate.  Of the library's kernels it knows those that the host paths
// under test depend on; the others do nothing.
#pragma once

#include <atomic>
#include <cstddef>

#include <hip/hip_runtime_api.h>

namespace fake {

void* device_alloc(size_t bytes);       // "device" memory, a range of its own
void device_free(void* p);
size_t queued();                        // operations that have not been executed
size_t stores_outside();                // kernel stores that lay past their allocation
// Queue an operation on a stream that ends only once `open` is set.
void queue_gate(hipStream_t s, const std::atomic<bool>* open);
void close_streams(bool closed);        // closed: nothing queued is executed
void set_last_error(hipError_t e);      // what an earlier call of this thread left behind

}  // namespace fake
