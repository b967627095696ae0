// Device blocks of destroyed contexts, kept for the next context of the process.
//
// A context's dictionary copies and Gram table are allocated when it is created and freed when it is destroyed.
// Programs that take one dictionary after another into use (an alternating dictionary update, a sweep) pay for
// that each time: mapping and clearing 288 MB for 6000 atoms costs 0.4 ms as long as the driver has cleared memory
// at hand and 7 ms when it does not, against 0.74 ms for computing the table itself.
//
// Bounded: at most POOL_BYTES per device stay here (a table of 11 000 atoms; larger blocks are freed at once, as
// allocators of the same process cannot take memory back from here), the oldest block leaves first; a block that no
// context has taken within POOL_AGE destroyed contexts is given back to the driver, and every block of the device is
// when an allocation of the library fails (the allocation is then tried again); bmpl_trim gives back all of them.
// Blocks are put here only after the device has been synchronised, so a block taken has no work in flight on any
// stream; a mutex serialises the threads.  The list is an array of fixed size: bmpl_destroy passes through here, and
// neither allocates nor throws.
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>

namespace bmpl {

constexpr size_t POOL_BYTES = (size_t)1 << 30;
constexpr int POOL_AGE = 8;
constexpr int POOL_BLOCKS = 64;

class BlockPool {
public:
    // A block of at least `bytes` on the current device `dev` (a kept one when its size is at most 1/8 larger).
    hipError_t take(int dev, void** out, size_t bytes, size_t* got) noexcept
    {
        *out = nullptr;
        if (bytes == 0) bytes = 1;
        {
            std::lock_guard<std::mutex> lk(mu_);
            int best = -1;
            for (int i = 0; i < n_; ++i)
                if (kept_[i].dev == dev && kept_[i].bytes >= bytes && kept_[i].bytes <= bytes + bytes / 8 &&
                    (best < 0 || kept_[i].bytes < kept_[best].bytes))
                    best = i;
            if (best >= 0) {
                *out = kept_[best].p;
                *got = kept_[best].bytes;
                erase(best);
                return hipSuccess;
            }
        }
        hipError_t e = hipMalloc(out, bytes);
        if (e == hipErrorOutOfMemory && drop(dev)) {
            (void)hipGetLastError();
            e = hipMalloc(out, bytes);
        }
        if (e != hipSuccess) (void)hipGetLastError();   // reported by the status: no later launch check may find it
        *got = bytes;
        return e;
    }

    // Take over a block (the device is synchronised and `dev` current).
    void put(int dev, void* p, size_t bytes) noexcept
    {
        std::lock_guard<std::mutex> lk(mu_);
        if (bytes > POOL_BYTES) {
            (void)hipFree(p);
            return;
        }
        if (n_ == POOL_BLOCKS) free_block(0);
        kept_[n_++] = {p, bytes, dev, 0};
        for (int i = 0; i < n_ && sum(dev) > POOL_BYTES;) {
            if (kept_[i].dev == dev) free_block(i);
            else ++i;
        }
    }

    // One more context of `dev` was destroyed: blocks that have waited too long go back.
    void age(int dev) noexcept
    {
        std::lock_guard<std::mutex> lk(mu_);
        for (int i = 0; i < n_;) {
            if (kept_[i].dev == dev && ++kept_[i].age > POOL_AGE) free_block(i);
            else ++i;
        }
    }

    // Bytes kept for `dev`.
    size_t kept(int dev) noexcept
    {
        std::lock_guard<std::mutex> lk(mu_);
        return sum(dev);
    }

    // Give every block of `dev` (-1: of every device) back; true if there was one.
    bool drop(int dev) noexcept
    {
        std::lock_guard<std::mutex> lk(mu_);
        bool any = false;
        for (int i = 0; i < n_;) {
            if (dev < 0 || kept_[i].dev == dev) {
                free_block(i);
                any = true;
            } else {
                ++i;
            }
        }
        return any;
    }

private:
    struct Block { void* p; size_t bytes; int dev; int age; };
    std::mutex mu_;
    Block kept_[POOL_BLOCKS];     // the oldest first
    int n_ = 0;

    void erase(int i) noexcept
    {
        for (--n_; i < n_; ++i) kept_[i] = kept_[i + 1];
    }
    void free_block(int i) noexcept
    {
        (void)hipFree(kept_[i].p);
        erase(i);
    }
    size_t sum(int dev) const noexcept
    {
        size_t b = 0;
        for (int i = 0; i < n_; ++i) b += kept_[i].dev == dev ? kept_[i].bytes : 0;
        return b;
    }
};

// Never destroyed: the HIP runtime may be gone before a static destructor runs (the process's end frees all).
inline BlockPool& block_pool()
{
    static BlockPool* pool = new BlockPool;
    return *pool;
}

}  // namespace bmpl
