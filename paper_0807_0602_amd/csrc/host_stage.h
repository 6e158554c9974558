// Page-locked host memory that kernels read from and write to directly, for small transfers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

#include <mutex>

namespace scf {

// A copy between the device and pageable memory takes 24 us at 64 bytes and 43 at 64 KB; a kernel that
// writes to page-locked memory, the synchronisation that is needed anyway and a host copy into the
// caller's array take 13 and 17.  Beyond about 1 MB the host copy costs what it saves.
constexpr size_t kStageBytes = (size_t)1 << 20;

// The process's buffers of kStageBytes, which all contexts share: a call takes one for as long as it
// lasts (StageLease).  Allocated when calls first overlap that far, so that creating a context costs
// nothing and destroying one frees nothing: hipHostFree waits for the whole device (144 ms for a
// channel destroyed while another stream was that busy, 0.01 ms now).  At most kBuffers; a call that
// finds all of them taken copies instead.  The last context gives back all but the first, which stays
// with the process; nothing is freed at its exit, when the HIP runtime may be gone.
class StagePool {
    static constexpr int kBuffers = 8;
    struct Buffer {
        char* p = nullptr;
        bool taken = false;
    };
    std::mutex mu;
    Buffer buffers[kBuffers];
    int contexts = 0;

    // Allocating and freeing are legal while a stream of the caller's is being captured in this mode.
    struct Relaxed {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
        ~Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    };

public:
    static StagePool& get() {
        static StagePool* pool = new StagePool;
        return *pool;
    }

    // NULL where every buffer is taken or page-locked memory is not to be had.
    char* take() {
        const std::lock_guard<std::mutex> hold(mu);
        Buffer* none = nullptr;
        for (Buffer& b : buffers) {
            if (b.p && !b.taken) {
                b.taken = true;
                return b.p;
            }
            if (!b.p && !none) none = &b;
        }
        if (!none) return nullptr;
        const Relaxed relaxed;
        void* p = nullptr;
        if (hipHostMalloc(&p, kStageBytes, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        none->p = static_cast<char*>(p);
        none->taken = true;
        return none->p;
    }

    void give(char* p) {
        const std::lock_guard<std::mutex> hold(mu);
        for (Buffer& b : buffers)
            if (b.p == p) b.taken = false;
    }

    void enter() {
        const std::lock_guard<std::mutex> hold(mu);
        ++contexts;
    }

    void leave() {
        const std::lock_guard<std::mutex> hold(mu);
        if (--contexts > 0) return;
        for (Buffer& b : buffers)
            if (&b != buffers && b.p && !b.taken) {
                const Relaxed relaxed;
                (void)hipHostFree(b.p);
                b.p = nullptr;
            }
    }
};

// One call's buffer: `p` is NULL where `bytes` do not fit one or none is free; the transfer is then a
// copy.  The call says done() once it has waited for stream s; a call that fails before that waits here.
class StageLease {
    hipStream_t s;
    bool idle = false;

public:
    char* p = nullptr;

    StageLease(size_t bytes, hipStream_t stream) : s(stream) {
        if (bytes > 0 && bytes <= kStageBytes) p = StagePool::get().take();
    }
    StageLease(const StageLease&) = delete;
    StageLease& operator=(const StageLease&) = delete;
    ~StageLease() {
        if (!p) return;
        if (!idle) (void)hipStreamSynchronize(s);
        StagePool::get().give(p);
    }
    void done() { idle = true; }
};

// A context's part: threads may read from one context, so a read-out holds `mu` from its launch to the
// end of its host copy, whether it goes through a buffer or through the idle population buffer or
// activations, which other read-outs use too.
struct HostStage {
    std::mutex mu;

    HostStage() { StagePool::get().enter(); }
    HostStage(const HostStage&) = delete;
    HostStage& operator=(const HostStage&) = delete;
    ~HostStage() { StagePool::get().leave(); }
};

}  // namespace scf
