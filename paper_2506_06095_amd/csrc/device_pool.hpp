// Device memory of destroyed plans, kept for the next ones: allocating and freeing a plan's few blocks cost more than
// analysing a small mask (plan, forward and destroy for a new 1024 x 1024 mask: 121 us, with blocks kept 112).  Only blocks of
// up to 1 MB, 16 MB of them at most.  A block comes in when no launch uses it any more, so that whoever takes it may use
// it on any stream.  Allocating and freeing are the runtime's (0: done), which refuses both while a thread captures: a
// block that cannot be freed then stays here.
#pragma once
#include <cstddef>
#include <mutex>
#include <new>
#include <vector>

namespace smha {

class DevicePool {
  public:
    using Alloc = int (*)(void **, size_t);
    using Free = int (*)(void *);
    static constexpr size_t kBlockAtMost = (size_t)1 << 20, kAtMost = (size_t)16 << 20;

    DevicePool(Alloc alloc, Free free) : alloc_(alloc), free_(free) {}

    static size_t block_size(size_t bytes) {  // what a block for so many bytes has
        if (bytes > kBlockAtMost) return bytes;
        size_t n = (size_t)64 << 10;
        while (n < bytes) n *= 2;
        return n;
    }
    // a block that was not kept; if there is no memory, what is kept goes back to the device first
    int fresh(void **ptr, size_t bytes) {
        if (alloc_(ptr, bytes) == 0) return 0;
        {
            std::lock_guard<std::mutex> lock(mutex_);
            while (!blocks_.empty() && free_(blocks_.back().ptr) == 0) {
                kept_ -= blocks_.back().bytes;
                blocks_.pop_back();
            }
        }
        return alloc_(ptr, bytes);
    }
    int take(void **ptr, size_t bytes, int device) {  // (`device` is current)
        const size_t want = block_size(bytes);
        if (want <= kBlockAtMost) {
            std::lock_guard<std::mutex> lock(mutex_);
            for (size_t i = blocks_.size(); i-- > 0;)
                if (blocks_[i].device == device && blocks_[i].bytes == want) {
                    *ptr = blocks_[i].ptr;
                    blocks_[i] = blocks_.back();
                    blocks_.pop_back();
                    kept_ -= want;
                    return 0;
                }
        }
        return fresh(ptr, want);
    }
    // `idle`: no launch uses the block
    void give(void *ptr, size_t bytes, int device, bool idle) {
        const size_t have = block_size(bytes);
        if (idle && have <= kBlockAtMost) {
            std::lock_guard<std::mutex> lock(mutex_);
            if (kept_ + have <= kAtMost) {
                try {
                    blocks_.push_back({ptr, have, device});
                    kept_ += have;
                    return;
                } catch (const std::bad_alloc &) {
                }
            }
        }
        (void)free_(ptr);
    }

  private:
    struct Block { void *ptr; size_t bytes; int device; };
    const Alloc alloc_;
    const Free free_;
    std::mutex mutex_;
    std::vector<Block> blocks_;
    size_t kept_ = 0;
};

}  // namespace smha
