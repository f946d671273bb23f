// host_copy.hip -- pageable copies through pinned buffers and worker threads.
#include <hip/hip_runtime.h>
#include <sched.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "host_copy.hpp"

namespace lbm {

namespace {

constexpr int kWorkers = 8;
constexpr size_t kChunk = size_t(2) << 20;
// Copies of up to this many bytes go directly: the workers' threads, and for a process's first
// large copy the pinning, would take longer. ms, direct | workers (the pinning is 0.05 to 0.2 more):
//   to the device, array in the CPU's caches   5 MB 0.15 | 0.22   16 MB 0.45 | 0.54   32 MB 0.88 | 0.94   48 MB 1.56 | 1.34
//                  array in memory             8 MB 0.30 | 0.38   16 MB 0.58 | 0.58   24 MB 0.84 | 0.80   48 MB 1.67 | 1.42
//   to the host    5 MB 0.27 | 0.20    6 MB 0.33 | 0.24    16 MB 0.90 | 0.54    48 MB 2.77 | 1.33
// (to a fresh array of 48 MB 4.69 | 1.42; chunks of 1 MiB 48 MB 1.62, 512 KiB 2.30)
constexpr size_t least(hipMemcpyKind kind) { return kind == hipMemcpyHostToDevice ? size_t(20) << 20 : size_t(6) << 20; }

std::mutex g_mu;            // holders and the buffer
int g_holders = 0;
bool g_busy = false;        // one staged copy at a time; another thread's copy meanwhile goes directly
char *g_buf = nullptr;      // a chunk for each worker

int worker_count() {
    static const std::string quota = [] {   // this process's limit; a container sees its own group at the root
        char text[64] = "";
        if (FILE *f = fopen("/sys/fs/cgroup/cpu.max", "r")) {
            if (!fgets(text, sizeof text, f)) text[0] = 0;
            fclose(f);
        }
        return std::string(text);
    }();
    cpu_set_t set;
    return workers_for(sched_getaffinity(0, sizeof set, &set) == 0 ? CPU_COUNT(&set) : 1, quota.c_str());
}

// allocation and waits here leave a capture on another thread's stream alone
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// device dev is current while this lives, in the caller's thread too, whose own is then restored
struct CurrentDevice {
    int was = -1;
    hipError_t e;
    explicit CurrentDevice(int dev) {
        e = hipGetDevice(&was);
        if (e == hipSuccess && was != dev) e = hipSetDevice(dev);
        else was = -1;
    }
    ~CurrentDevice() {
        if (was >= 0) (void)hipSetDevice(was);
    }
};

// pinned memory, or nullptr with no error left behind
void *pinned(size_t bytes) {
    RelaxedCapture relaxed;
    void *p = nullptr;
    if (hipHostMalloc(&p, bytes, hipHostMallocPortable) == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
}

// takes the buffer (allocating it if missing), or returns false
bool take() {
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_busy || g_holders == 0) return false;
    if (!g_buf && !(g_buf = (char *)pinned(kWorkers * kChunk))) return false;
    g_busy = true;
    return true;
}

void give() {
    std::lock_guard<std::mutex> lk(g_mu);
    g_busy = false;
}

// device, managed and pinned memory is copied directly
bool pageable(const void *p) {
    hipPointerAttribute_t a{};
    const hipError_t e = hipPointerGetAttributes(&a, p);
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipErrorInvalidValue || (e == hipSuccess && a.type == hipMemoryTypeUnregistered);
}

bool capturing(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(s, &st) != hipSuccess || st != hipStreamCaptureStatusNone;
}

}  // namespace

int workers_for(int cpus, const char *cpu_max) {
    long long quota = 0, period = 0;
    if (sscanf(cpu_max, "%lld %lld", &quota, &period) == 2 && quota > 0 && period > 0)
        cpus = (int)std::min<long long>(cpus, quota / period);
    return std::max(1, std::min(kWorkers, cpus / 2));
}

void staging_hold() {
    std::lock_guard<std::mutex> lk(g_mu);
    ++g_holders;
}

void staging_release() {
    std::lock_guard<std::mutex> lk(g_mu);
    if (--g_holders > 0) return;
    if (g_buf) (void)hipHostFree(g_buf);
    g_buf = nullptr;
}

hipError_t copy_pageable(int dev, hipStream_t stream, void *dst, const void *src, size_t bytes, hipMemcpyKind kind) {
    const void *host = kind == hipMemcpyHostToDevice ? src : dst;
    const int n = bytes <= least(kind) ? 1 : worker_count();
    // (hipStreamPerThread names another stream in each worker, not ordered with the caller's)
    if (n < 2 || stream == hipStreamPerThread || capturing(stream) || !pageable(host) || !take())
        return hipMemcpyAsync(dst, src, bytes, kind, stream);
    std::atomic<size_t> next{0};
    std::atomic<int> err{(int)hipSuccess};
    auto work = [&](int w) {
        RelaxedCapture relaxed;
        char *const buf = g_buf + (size_t)w * kChunk;
        const CurrentDevice current(dev);
        hipError_t e = current.e;
        hipEvent_t ev = nullptr;
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        while (e == hipSuccess && err.load() == (int)hipSuccess) {
            const size_t at = next.fetch_add(kChunk);
            if (at >= bytes) break;
            const size_t len = std::min(kChunk, bytes - at);
            if (kind == hipMemcpyHostToDevice) {
                memcpy(buf, (const char *)src + at, len);
                e = hipMemcpyAsync((char *)dst + at, buf, len, kind, stream);
            } else {
                e = hipMemcpyAsync(buf, (const char *)src + at, len, kind, stream);
            }
            if (e == hipSuccess) e = hipEventRecord(ev, stream);
            if (e == hipSuccess) e = hipEventSynchronize(ev);
            else (void)hipStreamSynchronize(stream);   // the buffer may be in use
            if (e == hipSuccess && kind == hipMemcpyDeviceToHost) memcpy((char *)dst + at, buf, len);
        }
        if (e != hipSuccess) err.store((int)e);
        if (ev) (void)hipEventDestroy(ev);
    };
    std::vector<std::thread> threads;
    try {
        threads.reserve((size_t)n - 1);
        for (int w = 1; w < n; ++w) threads.emplace_back(work, w);
    } catch (...) {
        // fewer threads than asked for: the ones there are take all the chunks
    }
    work(0);
    for (std::thread &t : threads) t.join();
    give();
    return (hipError_t)err.load();
}

hipError_t read_block(hipStream_t stream, const void *block, size_t bytes, const BlockPart *parts, int n, void **pin,
                      size_t pin_bytes) {
    bool staged = bytes <= pin_bytes;
    for (int k = 0; k < n; ++k) staged = staged && (!parts[k].dst || pageable(parts[k].dst));
    if (staged && !*pin) staged = (*pin = pinned(pin_bytes)) != nullptr;
    hipError_t e = hipSuccess;
    if (staged) e = hipMemcpyAsync(*pin, block, bytes, hipMemcpyDeviceToHost, stream);
    for (int k = 0; k < n && !staged && e == hipSuccess; ++k)
        if (parts[k].dst)
            e = hipMemcpyAsync(parts[k].dst, (const char *)block + parts[k].at, parts[k].bytes, hipMemcpyDeviceToHost, stream);
    const hipError_t se = hipStreamSynchronize(stream);
    if (e == hipSuccess) e = se;
    for (int k = 0; k < n && staged && e == hipSuccess; ++k)
        if (parts[k].dst) memcpy(parts[k].dst, (const char *)*pin + parts[k].at, parts[k].bytes);
    return e;
}

}  // namespace lbm
