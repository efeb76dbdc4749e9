// Device memory of the launches' intermediate buffers: a memory pool of the
// library's own per device.
//
// hipMallocAsync's default pool returns what it holds to the system whenever
// the program waits for the GPU, and the next call maps its gigabytes again: a
// g g -> t tbar g g g call of 6001 events x 17 points took 836 ms after each
// synchronisation against 92 ms without.  This pool keeps up to kPoolKeep
// bytes across synchronisations while a handle is open.  The last one to be
// destroyed gives back what is free and, since its last calls may still be
// running, sets the bytes to keep to 0, so that the next synchronisation
// returns the rest.  What a call needs beyond kPoolKeep (from 5.4 10^6 events of
// g g -> t tbar g g in single precision on, whose records are one buffer) still
// goes back at every synchronisation (2^23 events x 2 points, 20 GB: 193.8 ms
// each when the GPU is waited for after every call, 192.9 queued).  Allocations
// and releases are stream-ordered, from any thread, as with the default pool.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <type_traits>

namespace mgrw {

constexpr uint64_t kPoolKeep = uint64_t(12) << 30;

struct work_pools {
    static constexpr int kDevices = 64;
    std::mutex mu;
    hipMemPool_t pool[kDevices] = {};
    long handles = 0;

    // The pool of the stream's device (the current one for the default stream);
    // null where there is none.
    hipMemPool_t of_stream(hipStream_t s) {
        int dev = -1;
        if (s && hipStreamGetDevice(s, &dev) != hipSuccess) {
            (void)hipGetLastError();
            s = nullptr;
        }
        if (!s && hipGetDevice(&dev) != hipSuccess) return nullptr;
        if (dev < 0 || dev >= kDevices) return nullptr;
        std::lock_guard<std::mutex> lock(mu);
        if (!pool[dev]) {
            hipMemPoolProps props = {};
            props.allocType = hipMemAllocationTypePinned;
            props.handleTypes = hipMemHandleTypeNone;
            props.location.type = hipMemLocationTypeDevice;
            props.location.id = dev;
            hipMemPool_t p = nullptr;
            if (hipMemPoolCreate(&p, &props) != hipSuccess) {
                (void)hipGetLastError();
                return nullptr;
            }
            keep(p, kPoolKeep);
            pool[dev] = p;
        }
        return pool[dev];
    }
    void handle_created() {
        std::lock_guard<std::mutex> lock(mu);
        if (handles++ > 0) return;
        for (hipMemPool_t p : pool)
            if (p) keep(p, kPoolKeep);
    }
    void handle_destroyed() {
        std::lock_guard<std::mutex> lock(mu);
        if (--handles > 0) return;
        for (hipMemPool_t p : pool) {
            if (!p) continue;
            keep(p, 0);
            if (hipMemPoolTrimTo(p, 0) != hipSuccess) (void)hipGetLastError();
        }
    }
    static void keep(hipMemPool_t p, uint64_t bytes) {
        if (hipMemPoolSetAttribute(p, hipMemPoolAttrReleaseThreshold, &bytes) != hipSuccess) (void)hipGetLastError();
    }
};
inline work_pools& pools() {
    // never destroyed (handles may outlive static objects) and nothing that throws
    static_assert(std::is_trivially_destructible<work_pools>::value, "no destructor at exit");
    static work_pools p;
    return p;
}

// Stream-ordered allocation for a launch on stream s, released with
// hipFreeAsync.  Under stream capture the default pool serves it, whose
// allocations become nodes of the graph.
inline hipError_t work_alloc(void** ptr, size_t bytes, hipStream_t s) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &capture) != hipSuccess) {
        (void)hipGetLastError();
        capture = hipStreamCaptureStatusActive;
    }
    hipMemPool_t p = capture == hipStreamCaptureStatusNone ? pools().of_stream(s) : nullptr;
    if (p) {
        hipError_t err = hipMallocFromPoolAsync(ptr, bytes, p, s);
        if (err == hipSuccess) return err;
        (void)hipGetLastError();
        // what the pool keeps may be what is missing
        if (hipMemPoolTrimTo(p, 0) != hipSuccess) (void)hipGetLastError();
        err = hipMallocFromPoolAsync(ptr, bytes, p, s);
        if (err == hipSuccess) return err;
        (void)hipGetLastError();   // the default pool may still have room
    }
    return hipMallocAsync(ptr, bytes, s);
}

}  // namespace mgrw
