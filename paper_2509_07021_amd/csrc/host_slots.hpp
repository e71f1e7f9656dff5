// host_slots.hpp -- pinned words through which a kernel hands a counted total to the host that waits for it.
// Host code only but for the layout of HostCount, which the kernels write.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <string.h>

#include <chrono>
#include <mutex>

namespace megs {

// One slot, in pinned coherent host memory: the sequence number is the one the host gave out, written last.
struct HostCount {
    uint32_t total;
    int32_t bad_lobes;
    uint32_t seq;
    uint32_t total2;  // of a compaction: kept lobes
    uint32_t pad[12];  // one slot per 64 bytes
};

// The slots: one 4 KiB block for the process, portable over devices, its 64 slots lent to one call each; a
// call that finds none, or whose stream is being captured, copies the words with the stream instead.
// Measured on the eager forward of 2,000 Gaussians: two copies to pageable memory and the
// synchronisation left the GPU idle for 100 us; the polled slot for 20 us.
class HostSlots {
public:
    HostCount* take(uint32_t* seq) {
        std::lock_guard<std::mutex> lock(mu_);
        if (!base_) allocate();
        if (n_free_ == 0) return nullptr;
        if (++seq_ == 0) ++seq_;
        *seq = seq_;
        return base_ + free_[--n_free_];
    }
    void give(HostCount* s) {
        std::lock_guard<std::mutex> lock(mu_);
        free_[n_free_++] = (int)(s - base_);
    }

private:
    static constexpr int kSlots = 64;

    // Another thread may be capturing a stream in global mode, where an allocation is refused unless this
    // thread asks for the relaxed mode. A refused allocation is tried again by the next call.
    void allocate() {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        void* p = nullptr;
        if (hipHostMalloc(&p, sizeof(HostCount) * kSlots,
                          hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess) {
            memset(p, 0, sizeof(HostCount) * kSlots);
            base_ = static_cast<HostCount*>(p);
            for (n_free_ = 0; n_free_ < kSlots; ++n_free_) free_[n_free_] = n_free_;
        } else {
            (void)hipGetLastError();
        }
        if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }

    std::mutex mu_;
    HostCount* base_ = nullptr;
    int free_[kSlots], n_free_ = 0;
    uint32_t seq_ = 0;
};

// One call's use of a slot: taken before the launches, waited for after them. A call that ends in between
// (a failed launch) waits for the stream before it gives the slot back; where that fails too, the slot is not
// lent again (a kernel might still write it).
class SlotUse {
public:
    SlotUse(HostSlots& pool, hipStream_t s) : pool_(pool), stream_(s) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cap) != hipSuccess)
            (void)hipGetLastError();
        else if (cap == hipStreamCaptureStatusNone)
            slot = pool.take(&seq);
    }
    ~SlotUse() {
        if (slot && hipStreamSynchronize(stream_) == hipSuccess) pool_.give(slot);
    }
    SlotUse(const SlotUse&) = delete;
    SlotUse& operator=(const SlotUse&) = delete;

    // Polls for a while (the wait is normally tens of microseconds), then waits for the stream.
    hipError_t wait(uint32_t* total, int32_t* bad_lobes, uint32_t* total2 = nullptr) {
        const auto t0 = std::chrono::steady_clock::now();
        bool there = false;
        while (!(there = __atomic_load_n(&slot->seq, __ATOMIC_ACQUIRE) == seq)) {
            for (int i = 0; i < 32; ++i) __builtin_ia32_pause();
            if (std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(2)) break;
        }
        if (!there) {
            const hipError_t e = hipStreamSynchronize(stream_);
            if (e != hipSuccess) return e;
            if (__atomic_load_n(&slot->seq, __ATOMIC_ACQUIRE) != seq) return hipErrorUnknown;
        }
        *total = slot->total;
        if (total2) *total2 = slot->total2;
        *bad_lobes = slot->bad_lobes;
        pool_.give(slot);
        slot = nullptr;
        return hipSuccess;
    }

    HostCount* slot = nullptr;  // null: there is none, or it has been given back
    uint32_t seq = 0;

private:
    HostSlots& pool_;
    hipStream_t stream_;
};

}  // namespace megs
