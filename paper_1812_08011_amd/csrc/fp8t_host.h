// Host-side helpers shared by the library's entry points.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include <atomic>
#include <mutex>

#include "fp8train.h"

namespace fp8t {

// Largest M, N or K a GEMM entry point accepts: the kernels index rows,
// columns and k in 32 bits and form tile and slab ends (up to 4096 past an
// index) without overflow.
constexpr int64_t kMaxGemmDim = INT32_MAX - 4096;

// Blocks of a grid-stride launch over `total` items, `per_block` per block
// and pass: enough to fill the chip, never beyond the grid's limit.
inline unsigned stride_blocks(int64_t total, int per_block) {
    const int64_t b = (total + per_block - 1) / per_block;
    return (unsigned)(b < 65536 ? (b > 0 ? b : 1) : 65536);
}

inline bool aligned(const void* p, uintptr_t a) {
    return ((uintptr_t)p % a) == 0;
}

// Status of the launch just enqueued.
inline int launch_status() {
    return hipGetLastError() == hipSuccess ? FP8T_OK : FP8T_EHIP;
}

// Integer value of an environment variable (tests and tuning overrides).
inline int env_int(const char* name, int dflt) {
    const char* v = getenv(name);
    return v ? atoi(v) : dflt;
}

// Compute units of the current device (cached per device).
inline int device_cus() {
    static std::mutex mu;
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    std::lock_guard<std::mutex> lk(mu);
    if (!cached[dev]) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return 0;
        cached[dev] = n;
    }
    return cached[dev];
}

// The current device, -1 on error.
inline int current_device() {
    int dev = 0;
    return hipGetDevice(&dev) == hipSuccess ? dev : -1;
}

// Resident workgroups per CU of a kernel on device `dev`, the current one,
// cached per device and kernel in a hash table whose entries are written under
// a lock, once, and read without it: a planner asks for every configuration on
// each call (a locked scan over some 200 entries and the device asked for each
// time: 2.0-2.6 us of an exact GEMM's call, now 1.1).
inline int kernel_occupancy(const void* fn, int threads, int dev) {
    struct Ent {
        std::atomic<const void*> fn;      // set last; null: free
        int dev, occ;
    };
    constexpr size_t kSlots = 1024, kFull = 3 * kSlots / 4;
    static Ent cache[kSlots];             // zero: static storage
    static std::mutex mu;
    static size_t n = 0;
    auto find = [&](size_t& i) {
        i = (size_t)(((((uintptr_t)fn >> 4) + (uintptr_t)dev * 131) * 0x9E3779B97F4A7C15ull) >> 54);
        for (;; i = (i + 1) % kSlots) {
            const void* f = cache[i].fn.load(std::memory_order_acquire);
            if (!f) return false;
            if (f == fn && cache[i].dev == dev) return true;
        }
    };
    size_t i;
    if (find(i)) return cache[i].occ;
    int occ = 0;
    if (dev < 0 || hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, threads, 0) != hipSuccess)
        return 0;
    std::lock_guard<std::mutex> lk(mu);
    if (!find(i) && n < kFull) {
        cache[i].dev = dev;
        cache[i].occ = occ;
        cache[i].fn.store(fn, std::memory_order_release);
        ++n;
    }
    return occ;
}

}  // namespace fp8t
