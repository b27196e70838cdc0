// Device memory of the library's handles and workspaces.
//
// dev_alloc / dev_free have the meaning of hipMalloc / hipFree, with freed
// blocks kept for the next request of the same size.  A program that builds
// one operator after another (a new gauge field per step) frees and allocates
// the same gigabytes over and over, and the driver clears freed memory before
// it hands it out again: on MI355X one build of a 32^3 x 64 operator
// (5.2 GB) stalled for 10 to 400 ms in hipMalloc, 75 to 160 ms on average,
// next to 4 ms of kernels.
//
// Rules that keep this safe:
//   * the device is waited for (as hipFree does) between the freeing of a
//     block and its next use, once for all blocks freed so far, so no work on
//     any stream still uses a block that is handed out again;
//   * a block goes back only to requests on the device it belongs to;
//   * at most 1/16 of a device's memory is kept (18 GB of 288 GB), the
//     longest-kept blocks are freed first, and everything kept is freed as
//     soon as no lattice handle exists, or when an allocation fails (which is
//     then tried again);
//   * destroying a handle waits for the device (dev_wait), as the hipFree calls
//     did: what a caller queued with the handle has run when it is gone;
//   * other allocators of the process cannot reach the kept blocks; a caller
//     that needs them back uses dev_release (cs_release_cached_memory);
//   * contents are not cleared, as with hipMalloc.
// All calls may be made from any thread.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace cs {

hipError_t dev_alloc(void** p, size_t bytes);
void dev_free(void* p);  // p may be null

// Waits for all work on the device that the block p (handed out, or null)
// belongs to.
void dev_wait(const void* p);

// Gives all kept blocks back.
void dev_release();

// Lattice handles alive (a handle is created / destroyed): blocks are kept
// only while there is one.
void dev_lattice_created();
void dev_lattice_destroyed();

}  // namespace cs
