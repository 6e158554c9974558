// Page-locked host memory that kernels read from and write to directly, for small transfers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

#include <cstring>
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

// FP64 fields of up to kWidenBytes each come as FP32, half the bytes, into the upper halves of the
// caller's arrays and are widened there in place; larger ones come as they are (two fields, us in FP32 and
// in FP64, into arrays in use and into fresh pages: 90000 nodes 81 and 96, 359 and 406; 819200 610 and 766,
// 3230 and 3890; 2621440 2200 and 2415, 11260 and 12540; 5242880 4820 and 4920, 23700 and 25200; 16777216
// 16060 and 15580, 78100 and 81680).
constexpr size_t kWidenBytes = (size_t)40 << 20;

// a[i] = the i-th of the n FP32 values in the upper half of a, for every i.  In order and eight at a time:
// what is written ends before the values that are still to be read.
inline void widen(double* a, size_t n) {
    const char* f = reinterpret_cast<const char*>(a) + sizeof(float) * n;
    size_t i = 0;
    for (; i + 8 <= n; i += 8) {
        float v[8];
        double d[8];
        std::memcpy(v, f + sizeof(float) * i, sizeof v);
        for (int j = 0; j < 8; ++j) d[j] = v[j];
        std::memcpy(a + i, d, sizeof d);
    }
    for (; i < n; ++i) {
        float v;
        std::memcpy(&v, f + sizeof(float) * i, sizeof v);
        a[i] = v;
    }
}

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
