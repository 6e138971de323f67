// A bounded store of host memory blocks that go from one user to the next.
#pragma once
#include <stddef.h>

#include <mutex>

namespace dba {

struct HostBlock {
    unsigned char *p = nullptr;
    size_t bytes = 0;
};

// Memory: allocate(bytes) (null if there is none) and release(pointer).  Both are taken to be expensive, and called
// without the lock held.  Safe with several threads.
template <typename Memory>
class HostBlocks {
public:
    static constexpr size_t kLeast = 64 * 1024, kMost = 1024 * 1024, kKeepBytes = 2 * kMost;
    // an empty block if there is none to be had: its user does without
    HostBlock get(size_t bytes) noexcept
    {
        HostBlock block;
        if (bytes > kMost) return block;
        {
            // the smallest one that is large enough
            std::lock_guard<std::mutex> hold(mutex_);
            int best = -1;
            for (int i = 0; i < n_; ++i)
                if (kept_[i].bytes >= bytes && (best < 0 || kept_[i].bytes < kept_[best].bytes)) best = i;
            if (best >= 0) return take(best);
        }
        size_t n = kLeast;
        while (n < bytes) n *= 2;
        block.p = static_cast<unsigned char *>(Memory::allocate(n));
        block.bytes = block.p ? n : 0;
        return block;
    }
    // Nobody uses the block any more.  At most kKeepBytes stay here: those that came last, which fit what is asked for now.
    void put(HostBlock block) noexcept
    {
        if (!block.p) return;
        HostBlock gone[kKeep];
        int n_gone = 0;
        {
            std::lock_guard<std::mutex> hold(mutex_);
            while (kept_bytes_ + block.bytes > kKeepBytes) gone[n_gone++] = take(0);
            kept_[n_++] = block;
            kept_bytes_ += block.bytes;
        }
        for (int i = 0; i < n_gone; ++i) Memory::release(gone[i].p);
    }

private:
    static constexpr int kKeep = (int)(kKeepBytes / kLeast);
    HostBlock take(int i)
    {
        const HostBlock block = kept_[i];
        for (--n_; i < n_; ++i) kept_[i] = kept_[i + 1];
        kept_bytes_ -= block.bytes;
        return block;
    }
    std::mutex mutex_;
    HostBlock kept_[kKeep];               // in the order in which they came
    int n_ = 0;
    size_t kept_bytes_ = 0;
};

}  // namespace dba
