// A bounded list of page-locked buffers that calls of any thread lease and give back.
// Host code only; the allocator is the caller's, so that it can be tested without a GPU.
#pragma once

#include <stddef.h>

#include <mutex>

namespace df {

class PinnedPool {
public:
    static constexpr size_t kSmallest = 256 * 1024;   // buffers are this times a power of two
    static constexpr size_t kLargest = 4 << 20;       // larger ones are not kept
    static constexpr size_t kTotal = 8 << 20;         // bytes kept at most
    static constexpr int kCount = 8;                  // buffers kept at most

    PinnedPool(void *(*alloc)(size_t), void (*release)(void *)) : alloc_(alloc), release_(release) {}

    // A buffer of at least `bytes` (its size in *cap), the smallest kept one that is large
    // enough or a new one; null without memory.
    void *take(size_t bytes, size_t *cap) {
        {
            std::lock_guard<std::mutex> lk(mu_);
            int best = -1;
            for (int i = 0; i < n_; ++i)
                if (kept_[i].cap >= bytes && (best < 0 || kept_[i].cap < kept_[best].cap)) best = i;
            if (best >= 0) {
                const Buffer b = kept_[best];
                drop(best);
                *cap = b.cap;
                return b.p;
            }
        }
        size_t c = kSmallest;
        while (c < bytes && c < kLargest) c *= 2;
        if (c < bytes) c = bytes;
        *cap = c;
        return alloc_(c);
    }

    // Keeps the buffer; the smallest ones make room (a larger one serves their calls too).
    void give(void *p, size_t cap) {
        void *out[kCount + 1];
        int n_out = 0;
        {
            std::lock_guard<std::mutex> lk(mu_);
            bool keep = cap <= kLargest;
            while (keep && (n_ == kCount || total_ + cap > kTotal)) {
                int least = 0;
                for (int i = 1; i < n_; ++i)
                    if (kept_[i].cap < kept_[least].cap) least = i;
                if (kept_[least].cap >= cap) keep = false;
                else {
                    out[n_out++] = kept_[least].p;
                    drop(least);
                }
            }
            if (keep) {
                kept_[n_++] = {p, cap};
                total_ += cap;
            } else out[n_out++] = p;
        }
        for (int i = 0; i < n_out; ++i) release_(out[i]);
    }

private:
    struct Buffer {
        void *p;
        size_t cap;
    };
    void drop(int i) {
        total_ -= kept_[i].cap;
        kept_[i] = kept_[--n_];
    }
    void *(*alloc_)(size_t);
    void (*release_)(void *);
    std::mutex mu_;
    Buffer kept_[kCount];
    int n_ = 0;
    size_t total_ = 0;
};

}  // namespace df
