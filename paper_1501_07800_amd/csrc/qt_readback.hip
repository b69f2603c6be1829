// The pools of pinned slots behind ReadBack, and its kernel.
#include "qt_readback.h"

#include <chrono>

namespace qt {

__global__ __launch_bounds__(1024) void k_publish(const int32_t* __restrict__ words, int64_t n, HostSlot* slot,
                                                  uint32_t seq) {
    publish_words(words, n, slot, seq);
}

typedef std::pair<HostSlot*, HostSlot*> SlotPair;   // (host address, device address)
static std::mutex g_slot_mu;
static std::vector<SlotPair> g_small, g_large;      // free slots
constexpr size_t kLargeKept = 8;                    // free large slots kept (256 KiB each)
static uint32_t g_seq = 0;

static size_t slot_bytes(int64_t words) { return (sizeof(HostSlot) + words * sizeof(int32_t) + 63) & ~size_t(63); }

static SlotPair pinned(size_t bytes) {
    void *h = nullptr, *d = nullptr;
    QT_HIP(hipHostMalloc(&h, bytes, hipHostMallocCoherent | hipHostMallocPortable | hipHostMallocMapped));
    QT_HIP(hipHostGetDevicePointer(&d, h, 0));
    return {(HostSlot*)h, (HostSlot*)d};
}

ReadBack::ReadBack(int64_t n) : n_(n) {
    if (n > kLargeSlotWords) return;
    std::lock_guard<std::mutex> lk(g_slot_mu);
    auto& pool = n <= kSlotWords ? g_small : g_large;
    if (pool.empty()) {
        if (n <= kSlotWords) {
            constexpr int kChunk = 16;
            const size_t each = slot_bytes(kSlotWords);
            const SlotPair p = pinned(kChunk * each);
            for (int i = 0; i < kChunk; ++i)
                pool.emplace_back((HostSlot*)((char*)p.first + i * each), (HostSlot*)((char*)p.second + i * each));
        } else {
            pool.push_back(pinned(slot_bytes(kLargeSlotWords)));
        }
    }
    slot_ = pool.back().first;
    dslot_ = pool.back().second;
    pool.pop_back();
    if (++g_seq == 0) ++g_seq;   // 0 never marks a publication
    seq_ = g_seq;
    __atomic_store_n(&slot_->flag, 0u, __ATOMIC_RELAXED);
}

ReadBack::~ReadBack() {
    if (!slot_) return;
    std::lock_guard<std::mutex> lk(g_slot_mu);
    if (n_ <= kSlotWords)
        g_small.emplace_back(slot_, dslot_);
    else if (g_large.size() < kLargeKept)
        g_large.emplace_back(slot_, dslot_);
    else
        (void)hipHostFree(slot_);
}

void ReadBack::publish(const int32_t* words, hipStream_t s) {
    if (!slot_) {
        copy_.resize(n_);
        QT_HIP(hipMemcpyAsync(copy_.data(), words, n_ * sizeof(int32_t), hipMemcpyDeviceToHost, s));
        return;
    }
    k_publish<<<1, n_ <= kSlotWords ? 64 : 1024, 0, s>>>(words, n_, dslot_, seq_);
    QT_LAUNCH("k_publish");
}

const int32_t* ReadBack::wait(hipStream_t s) {
    if (!slot_) {
        QT_HIP(hipStreamSynchronize(s));
        return copy_.data();
    }
    // Spin for a while (checking the stream now and then, so that a failed
    // launch ends the wait with its error), then leave the waiting to the
    // runtime: there may be any amount of earlier work on the stream.
    const auto t0 = std::chrono::steady_clock::now();
    for (uint64_t it = 1; __atomic_load_n(&slot_->flag, __ATOMIC_ACQUIRE) != seq_; ++it) {
        if ((it & 4095) != 0) continue;
        const hipError_t e = hipStreamQuery(s);
        if (e != hipSuccess && e != hipErrorNotReady) hip_check(e, "read-back");
        if (e == hipSuccess || std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(20)) {
            QT_HIP(hipStreamSynchronize(s));
            if (__atomic_load_n(&slot_->flag, __ATOMIC_ACQUIRE) != seq_)
                fail(QT_ERR_DEVICE, "read-back: the words were not published");
            break;
        }
    }
    return slot_->words;
}

}  // namespace qt
