// Host-side checks of the copies between pageable memory and the device (csrc/host_copy.hip).
// The HIP runtime calls it makes are defined here: a copy is a memcpy that notes the calling
// thread, streams are names, and each thread has its own current device, so no GPU is used.
// usage: copy_driver CHECK; exits 0 when every expectation of that check holds.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <string.h>

#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "host_copy.hpp"

using namespace lbm;

namespace {

std::mutex mu;
std::map<std::thread::id, int> copies;   // copies enqueued, by thread
bool fail_pinned = false;                // pinned allocations fail
const void *device_memory = nullptr;     // an address that is device memory; all others are pageable
int strict_allocations = 0;              // those made while a capture on another thread would break
thread_local hipStreamCaptureMode capture_mode = hipStreamCaptureModeGlobal;
thread_local int device = 0;
thread_local hipError_t last_error = hipSuccess;

hipError_t note(hipError_t e) {
    if (e != hipSuccess) last_error = e;
    return e;
}

int failures = 0;
#define EXPECT(cond)                                                                    \
    do {                                                                                \
        if (!(cond)) {                                                                  \
            fprintf(stderr, "expectation failed: %s (line %d)\n", #cond, __LINE__);     \
            ++failures;                                                                 \
        }                                                                               \
    } while (0)

}  // namespace

extern "C" {

hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *mode) {
    std::swap(*mode, capture_mode);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
    strict_allocations += capture_mode != hipStreamCaptureModeRelaxed;
    if (fail_pinned) return note(hipErrorOutOfMemory);
    *p = malloc(bytes);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    free(p);
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    if (p != device_memory) return note(hipErrorInvalidValue);
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
    *st = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = device;
    return hipSuccess;
}
hipError_t hipSetDevice(int d) {
    device = d;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = (hipEvent_t)malloc(1);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) {
    free((void *)e);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t bytes, hipMemcpyKind, hipStream_t) {
    {
        std::lock_guard<std::mutex> lk(mu);
        ++copies[std::this_thread::get_id()];
    }
    memcpy(dst, src, bytes);
    return hipSuccess;
}

}  // extern "C"

namespace {

// copies 64 MiB and a ragged end both ways and compares every byte; returns the threads that enqueued
size_t round_trip(hipStream_t stream) {
    const size_t n = (size_t(64) << 20) + 12345;
    std::vector<unsigned char> a(n), b(n), c(n);
    for (size_t k = 0; k < n; ++k) a[k] = (unsigned char)(k * 2654435761u >> 13);
    copies.clear();
    EXPECT(copy_pageable(0, stream, b.data(), a.data(), n, hipMemcpyHostToDevice) == hipSuccess);
    EXPECT(copy_pageable(0, stream, c.data(), b.data(), n, hipMemcpyDeviceToHost) == hipSuccess);
    EXPECT(a == c);
    return copies.size();
}

// two parts of a block of 1000 bytes, with and without pinned memory of pin_bytes; returns the copies made
int read_parts(size_t pin_bytes, void **pin, bool to_device = false) {
    std::vector<char> block(1000);
    for (size_t k = 0; k < block.size(); ++k) block[k] = (char)(k * 7);
    std::vector<char> a(40, 'x'), b(600, 'x');
    const BlockPart parts[] = {{a.data(), 0, a.size()}, {nullptr, 40, 360}, {b.data(), 400, b.size()}};
    device_memory = to_device ? b.data() : nullptr;
    copies.clear();
    EXPECT(read_block((hipStream_t) nullptr, block.data(), block.size(), parts, 3, pin, pin_bytes) == hipSuccess);
    EXPECT(!memcmp(a.data(), block.data(), a.size()) && !memcmp(b.data(), block.data() + 400, b.size()));
    return copies[std::this_thread::get_id()];
}

}  // namespace

int main(int argc, char **argv) {
    const std::string check = argc > 1 ? argv[1] : "";
    staging_hold();
    if (check == "data") {
        (void)round_trip((hipStream_t) nullptr);
    } else if (check == "worth_the_threads") {
        // one direct copy up to the sizes from which the workers are faster, several beyond
        std::vector<char> a(size_t(21) << 20), b(a.size());
        const struct { size_t mib; hipMemcpyKind kind; bool direct; } cases[] = {
            {1, hipMemcpyHostToDevice, true}, {5, hipMemcpyHostToDevice, true}, {20, hipMemcpyHostToDevice, true},
            {21, hipMemcpyHostToDevice, false}, {1, hipMemcpyDeviceToHost, true}, {6, hipMemcpyDeviceToHost, true},
            {7, hipMemcpyDeviceToHost, false}};
        for (const auto &c : cases) {
            copies.clear();
            EXPECT(copy_pageable(0, (hipStream_t) nullptr, b.data(), a.data(), c.mib << 20, c.kind) == hipSuccess);
            int n = 0;
            for (const auto &t : copies) n += t.second;
            EXPECT((n == 1) == c.direct);
        }
    } else if (check == "quota") {
        // half the CPUs, of the affinity mask or of the control group's quota, eight at most
        EXPECT(workers_for(16, "max 100000\n") == 8 && workers_for(256, "1600000 100000\n") == 8);
        EXPECT(workers_for(256, "400000 100000\n") == 2 && workers_for(256, "250000 100000\n") == 1);
        EXPECT(workers_for(4, "") == 2 && workers_for(1, "max 100000\n") == 1 && workers_for(6, "garbage") == 3);
        EXPECT(workers_for(64, "0 0\n") == 8 && workers_for(64, "50000 100000\n") == 1);
    } else if (check == "per_thread_stream") {
        // that handle names another stream in every thread: only the caller's is the one meant
        EXPECT(round_trip(hipStreamPerThread) == 1);
        EXPECT(copies.count(std::this_thread::get_id()) == 1);
    } else if (check == "current_device") {
        // the caller's current device is the same afterwards, whichever device is copied to
        for (int current : {0, 1}) {
            device = current;
            (void)round_trip((hipStream_t) nullptr);
            EXPECT(device == current);
        }
    } else if (check == "block") {
        void *pin = nullptr;
        EXPECT(read_parts(999, &pin) == 2 && !pin);    // larger than the pinned memory: part by part
        EXPECT(read_parts(1000, &pin) == 1 && pin);
        EXPECT(read_parts(1000, &pin) == 1);
        (void)hipHostFree(pin);
    } else if (check == "block_to_device") {
        // the host does not write to device memory: part by part
        void *pin = nullptr;
        EXPECT(read_parts(1000, &pin, true) == 2);
        (void)hipHostFree(pin);
    } else if (check == "no_pinned_memory") {
        // everything is copied directly, and no error is left behind
        fail_pinned = true;
        void *pin = nullptr;
        EXPECT(read_parts(1 << 20, &pin) == 2 && !pin);
        EXPECT(round_trip((hipStream_t) nullptr) == 1);
    } else if (check == "capture_mode") {
        // pinned memory is allocated in the relaxed capture mode, the thread's own is restored
        void *pin = nullptr;
        (void)read_parts(1000, &pin);
        (void)hipHostFree(pin);
        (void)round_trip((hipStream_t) nullptr);
        EXPECT(strict_allocations == 0 && capture_mode == hipStreamCaptureModeGlobal);
    } else {
        fprintf(stderr, "unknown check\n");
        return 2;
    }
    staging_release();
    EXPECT(last_error == hipSuccess);
    if (!failures) printf("copy driver ok\n");
    return failures ? 1 : 0;
}
