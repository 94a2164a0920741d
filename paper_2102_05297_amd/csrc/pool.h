// Memory and streams kept between handles.
//
// A program that opens one session, batch or model after another on a space
// pays the driver for every buffer: on MI355X a hipHostMalloc takes 20 to 50
// us, a hipHostFree 20 to 270 us, a hipMalloc and hipFree 15 to 40 us each
// (more for large blocks), a stream 50 us and 40 more to destroy (12 ms the
// process's first).  Released blocks and streams are therefore kept for the next
// handle.
//
//   - Bounded: at most kDeviceCap bytes of device memory per GPU, kPinnedCap
//     bytes of pinned host memory and kStreamCap streams are kept.  A block that
//     would exceed its bound makes the ones kept longest go back to the driver
//     first; everything kept goes back when an allocation fails (which is then
//     tried again).
//   - Given back: the pool lives as long as some space does.  When the last
//     space is destroyed, everything kept is returned to the driver, and on
//     request (cgs_release_memory) at any time.
//   - Threads: every call locks the pool.
//   - Streams: a block or stream is put back only once the work that used it
//     has finished (the caller has synchronised its stream), so the next
//     holder may use it on any stream.  Contents are unspecified.
// Blocks are sized in classes, so that handles of similar spaces share them.
//
// Measured: 64 sessions and their batch around 64 runs of 150 tests on 7,616
// configurations 56 -> 5.2 ms; one session around 17 steps 498 -> 340 us;
// loading and closing a perceptron model of 4.0M configurations 2.4 -> 1.6
// ms.  A program that keeps no space open pays what it paid before.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace cgs {
namespace pool {

constexpr size_t kDeviceCap = (size_t)1 << 30;
constexpr size_t kPinnedCap = (size_t)16 << 20;
constexpr size_t kStreamCap = 8;

// One more / one less live space; the last one empties the pool.
void attach();
void detach();

// Returns everything kept to the driver.
void release();

// A block of at least `bytes` on the current device.
hipError_t device_get(void **p, size_t bytes);
void device_put(void *p);
// Pinned, mapped, coherent host memory and its device address.
hipError_t pinned_get(void **host, void **dev, size_t bytes);
void pinned_put(void *host);
// A non-blocking stream of default priority on the current device.
hipError_t stream_get(hipStream_t *s);
void stream_put(hipStream_t s);

} // namespace pool
} // namespace cgs
