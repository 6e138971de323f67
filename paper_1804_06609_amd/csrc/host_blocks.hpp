// A bounded store of host memory blocks that go from one user to the next.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <string.h>

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
        for (bool settled = false;; settled = true) {
            {
                // the smallest one that is large enough
                std::lock_guard<std::mutex> hold(mutex_);
                int best = -1;
                for (int i = 0; i < n_; ++i)
                    if (kept_[i].bytes >= bytes && (best < 0 || kept_[i].bytes < kept_[best].bytes)) best = i;
                if (best >= 0) return take(best);
            }
            if (settled) break;
            settle();
        }
        size_t n = kLeast;
        while (n < bytes) n *= 2;
        block.p = static_cast<unsigned char *>(Memory::allocate(n));
        block.bytes = block.p ? n : 0;
        return block;
    }
    // Somebody still writes to the block's first n words: nobody does any more once each of them is `last` in the bits of `mask`.  Looked
    // at whenever blocks come and go; nothing waits, and a block whose words never come is left alone.
    void put_when(HostBlock block, uint32_t n, uint32_t last, uint32_t mask) noexcept
    {
        if (!block.p) return;
        {
            std::lock_guard<std::mutex> hold(mutex_);
            const Awaited a = {waiting_, n, last, mask};
            memcpy(note_of(block), &a, sizeof(a));
            waiting_ = block;
        }
        settle();
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
    // Blocks that are waited for form a list whose links lie at their ends, where nobody writes.
    struct Awaited {
        HostBlock next;
        uint32_t n, last, mask;
    };
    static unsigned char *note_of(HostBlock block) { return block.p + block.bytes - sizeof(Awaited); }
    static bool come(HostBlock block, const Awaited &a)
    {
        const uint32_t *words = reinterpret_cast<const uint32_t *>(block.p);
        for (uint32_t i = 0; i < a.n; ++i)
            if ((__atomic_load_n(words + i, __ATOMIC_RELAXED) & a.mask) != a.last) return false;
        return true;
    }
    // the blocks whose words have come go to the others
    void settle()
    {
        HostBlock ready;
        {
            std::lock_guard<std::mutex> hold(mutex_);
            HostBlock left, block = waiting_;
            while (block.p) {
                Awaited a;
                memcpy(&a, note_of(block), sizeof(a));
                HostBlock &list = come(block, a) ? ready : left;
                memcpy(note_of(block), &list, sizeof(HostBlock));
                list = block;
                block = a.next;
            }
            waiting_ = left;
        }
        while (ready.p) {
            const HostBlock block = ready;
            memcpy(&ready, note_of(block), sizeof(HostBlock));
            put(block);
        }
    }
    HostBlock take(int i)
    {
        const HostBlock block = kept_[i];
        for (--n_; i < n_; ++i) kept_[i] = kept_[i + 1];
        kept_bytes_ -= block.bytes;
        return block;
    }
    std::mutex mutex_;
    HostBlock waiting_;                   // the first of those that are waited for
    HostBlock kept_[kKeep];               // in the order in which they came
    int n_ = 0;
    size_t kept_bytes_ = 0;
};

}  // namespace dba
