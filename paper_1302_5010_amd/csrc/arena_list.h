// The slot blocks' arena: a list of chunks of device memory.  Plain C++ apart from the function attributes.
#pragma once

#ifdef __HIPCC__
#define BMPL_HOST_DEVICE __host__ __device__
#else
#define BMPL_HOST_DEVICE
#endif

namespace bmpl {

// Device arena of the per-signal slot blocks: a list of chunks viewed as one range of doubles.  Blocks
// are handed out by bumping `top` (a block never straddles two chunks); a signal whose active set
// outgrows its block takes a larger one and copies its state over.  The arena is reset for every solve.
constexpr int ARENA_CHUNKS = 32;
struct Arena {
    int n_act[2];                 // running-signal counts of the two running lists (read back with the rest)
    unsigned long long top;       // doubles handed out in this solve (offset in the chunk list)
    unsigned long long starved;   // block requests that found no room (the host adds a chunk)
    unsigned long long reserve;   // doubles the running signals may request during the next iterations
    unsigned long long grow_base; // offset of the blocks the last stop test placed for the grow list
    int nchunks;
    int pad_;
    double* base[ARENA_CHUNKS];
    unsigned long long start[ARENA_CHUNKS];   // offset of each chunk in the list (start[c+1] = start[c] + size[c])
    unsigned long long size[ARENA_CHUNKS];    // doubles
};

// One chunk of the list.  The host enqueues it by value: the list it writes itself may get the next chunk before the
// device has taken this one over (the host loop runs an iteration ahead), so the device never reads the host's list.
struct ArenaChunk {
    int index;
    double* base;
    unsigned long long start, size;
};

// The chunk of `size` doubles at `p` that comes next in the list.
inline ArenaChunk arena_next(const Arena& A, double* p, unsigned long long size)
{
    const int k = A.nchunks;
    return {k, p, k ? A.start[k - 1] + A.size[k - 1] : 0ull, size};
}

// Take a chunk over: its entry, then the count that makes it visible.
BMPL_HOST_DEVICE inline void arena_put(Arena& A, const ArenaChunk& c)
{
    A.base[c.index] = c.base;
    A.start[c.index] = c.start;
    A.size[c.index] = c.size;
    A.nchunks = c.index + 1;
}

}  // namespace bmpl
