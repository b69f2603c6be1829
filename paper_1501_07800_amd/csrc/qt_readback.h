// Reading words back from the device without a device-to-host copy and a
// stream synchronization (together 25-40 us on this machine before the host
// goes on): a kernel writes the words into pinned, host-coherent memory and
// then releases a sequence number there at system scope; the host spins on
// that word (about 8 us from the kernel's end).
#pragma once
#include "qt_internal.h"

namespace qt {

constexpr int64_t kSlotWords = 128;             // words of an ordinary slot
constexpr int64_t kLargeSlotWords = 1 << 16;    // of a large one; more go through a copy

struct alignas(64) HostSlot {
    uint32_t flag;
    int32_t pad[15];
    int32_t words[1];   // kSlotWords or kLargeSlotWords
};

// Called by every thread of one workgroup: n words into the slot, then the
// sequence number.
__device__ __forceinline__ void publish_words(const int32_t* words, int64_t n, HostSlot* slot, uint32_t seq) {
    for (int64_t t = threadIdx.x; t < n; t += blockDim.x) slot->words[t] = words[t];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(&slot->flag, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One read-back of n words: a pinned slot, taken from a pool and given back on
// scope exit. Nothing may throw between publish() and wait().
class ReadBack {
  public:
    explicit ReadBack(int64_t n);
    ~ReadBack();
    ReadBack(const ReadBack&) = delete;
    ReadBack& operator=(const ReadBack&) = delete;
    HostSlot* device_slot() const { return dslot_; }   // for a kernel that publishes by itself (n <= kSlotWords)
    uint32_t seq() const { return seq_; }
    void publish(const int32_t* words, hipStream_t s);   // queues it on s
    // Waits for the publication queued on s. The words stay valid as long as
    // this object.
    const int32_t* wait(hipStream_t s);

  private:
    int64_t n_;
    HostSlot* slot_ = nullptr;
    HostSlot* dslot_ = nullptr;
    uint32_t seq_ = 0;
    std::vector<int32_t> copy_;   // n_ > kLargeSlotWords
};

}  // namespace qt
