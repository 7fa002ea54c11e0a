// The count of live systems after a COCG step, from the device to the host.
#pragma once

#include <atomic>
#include <chrono>
#include <mutex>

#include "common.hpp"

namespace chaff {

// One page of pinned host memory per process, 64 slots: a solve takes a slot for
// its duration and gives it back once its stream has drained, also where it ends
// in an error (only a stream that fails itself keeps its slot, so that nothing
// late can be taken for another call's count).  Allocating per call would make
// every solve wait for every stream of the device when the memory is freed.
class FlagPage {
public:
    uint64_t* take(int& slot) {
        std::call_once(once_, [this] {
            void* m = nullptr;
            if (hipHostMalloc(&m, SLOTS * 64, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) ==
                hipSuccess)
                page_ = static_cast<char*>(m);
            else
                (void)hipGetLastError();
        });
        if (!page_) return nullptr;
        uint64_t free = free_.load();
        while (free) {
            const int s = __builtin_ctzll(free);
            if (free_.compare_exchange_weak(free, free & ~(1ull << s))) {
                slot = s;
                return reinterpret_cast<uint64_t*>(page_ + 64 * s);
            }
        }
        return nullptr;
    }
    void give(int slot) { free_.fetch_or(1ull << slot); }

private:
    static constexpr int SLOTS = 64;
    std::once_flag once_;
    char* page_ = nullptr;
    std::atomic<uint64_t> free_{~0ull};
};
inline FlagPage g_flag_page;

// The device writes sequence number << 32 | count to the slot and the host reads it
// there: a copy to pageable memory with its two waits held the next launch back by
// 45 us a step (100,000 wires x 8 waves 5.88 -> 5.63 ms; 12,000 x 8 2.26 -> 1.99).
// Without a slot (none free, or no pinned memory) the count is copied.
struct StepFlag {
    uint64_t* p = nullptr;
    uint32_t seq = 0;
    int slot = -1;
    hipStream_t st;

    explicit StepFlag(hipStream_t stream) : st(stream) {}
    StepFlag(const StepFlag&) = delete;
    StepFlag& operator=(const StepFlag&) = delete;
    ~StepFlag() {   // a solve that returned early may have steps in flight
        if (!p) return;
        if (hipStreamSynchronize(st) == hipSuccess)
            give();
        else
            (void)hipGetLastError();
    }
    void take() {
        if (!p && (p = g_flag_page.take(slot))) __atomic_store_n(p, 0, __ATOMIC_RELEASE);
    }
    // the caller's stream has drained
    void give() {
        if (p) g_flag_page.give(slot);
        p = nullptr;
    }
    bool read(int32_t& n) const {
        const uint64_t v = __atomic_load_n(p, __ATOMIC_ACQUIRE);
        n = (int32_t)(uint32_t)v;
        return (uint32_t)(v >> 32) == seq;
    }
    // the count of the step launched last; ends with the stream's work, in order or in error
    chaff_status wait(const int32_t* counter, int32_t& n) const {
        if (!p) {
            CHAFF_HIP(hipMemcpyAsync(&n, counter, sizeof(int32_t), hipMemcpyDeviceToHost, st));
            CHAFF_HIP(hipStreamSynchronize(st));
            return CHAFF_OK;
        }
        // the stream is asked only now and then: each query submits work of its own,
        // which held a run of 1 ms kernels back by 3%
        for (auto asked = std::chrono::steady_clock::now();;) {
            for (int i = 0; i < 1024; ++i) {
                if (read(n)) return CHAFF_OK;
                __builtin_ia32_pause();   // the core's other thread runs meanwhile
            }
            const auto now = std::chrono::steady_clock::now();
            if (now - asked < std::chrono::milliseconds(20)) continue;
            asked = now;
            const hipError_t e = hipStreamQuery(st);
            if (e == hipErrorNotReady) {
                (void)hipGetLastError();
                continue;
            }
            CHAFF_HIP(e);
            if (read(n)) return CHAFF_OK;
            return fail(CHAFF_EHIP, "a COCG step ended without its count");
        }
    }
};

}  // namespace chaff
