// Page-locked host memory that kernels read from and write to directly, for small transfers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

#include <mutex>

namespace scf {

// One per context, allocated with it and freed with it.  A copy between the device and pageable
// memory takes 24 us at 64 bytes and 43 at 64 KB; a kernel that writes here, the synchronisation that
// is needed anyway and a host copy into the caller's array take 13 and 17.  Beyond about 1 MB the host
// copy costs what it saves.  `p` is NULL where the memory was not to be had; transfers are then copies.
// Threads may read from one context: a read-out holds `mu` from its launch to the end of its host copy,
// whether it goes through this memory or through the idle population buffer or activations, which other
// read-outs use too.
constexpr size_t kStageBytes = (size_t)1 << 20;

struct HostStage {
    char* p = nullptr;
    size_t bytes = 0;
    std::mutex mu;

    HostStage() = default;
    HostStage(const HostStage&) = delete;
    HostStage& operator=(const HostStage&) = delete;
    ~HostStage() {
        if (p) (void)hipHostFree(p);
    }

    void reserve(size_t n) {
        if (p || n == 0) return;
        if (hipHostMalloc(reinterpret_cast<void**>(&p), n, hipHostMallocDefault) == hipSuccess) {
            bytes = n;
        } else {
            p = nullptr;
            (void)hipGetLastError();
        }
    }
    bool holds(size_t n) const { return n <= bytes; }
};

}  // namespace scf
