// host_copy.hpp -- copies between the caller's pageable memory and the device.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace lbm {

// Copies `bytes` between pageable host memory and device `dev` on `stream`, one of that device.
// The caller's current device stays as it is. Copies of more than 20 MiB to the device and 6 MiB to
// the host are complete on return; smaller ones, those of memory that is not pageable, those on
// hipStreamPerThread and those into a capture go to hipMemcpyAsync. The runtime's own copy of
// pageable memory goes through one thread, 18 GB/s to the host (10 into fresh arrays) and 29 to the
// device from memory; here worker threads take turns on the stream, each with a pinned 2 MiB of its
// own, so that one's transfer overlaps the others' copies (and the page faults of a fresh array):
// 35 GB/s either way.
hipError_t copy_pageable(int dev, hipStream_t stream, void *dst, const void *src, size_t bytes, hipMemcpyKind kind);

// Worker threads for `cpus` CPUs of the affinity mask under a control group's quota, the text of its
// cpu.max ("max" or microseconds, then the period; "" without one).
int workers_for(int cpus, const char *cpu_max);

// The pinned buffer is shared by all contexts of a process, 16 MiB; it is freed when the last
// holder lets go.
void staging_hold();
void staging_release();

// Reads parts of one device block back and waits for them. A block of up to pin_bytes comes in one
// copy into pinned memory at *pin (allocated when it is null; the caller frees it with hipHostFree)
// and is handed out from there. Without that memory, for larger blocks, and where a part goes to
// device, managed or pinned memory, each part is copied directly.
struct BlockPart {
    void *dst;          // nullptr: not wanted
    size_t at, bytes;   // its place in the block
};
hipError_t read_block(hipStream_t stream, const void *block, size_t bytes, const BlockPart *parts, int n, void **pin,
                      size_t pin_bytes);

}  // namespace lbm
