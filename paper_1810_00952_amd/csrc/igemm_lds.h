// What the contraction kernels with direct global -> LDS loads share: descriptors, the K loop's barrier.
#pragma once
#include "device_utils.h"

namespace rl {

namespace {

typedef __amdgpu_buffer_rsrc_t rsrc_t;
#define RL_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

__device__ __forceinline__ rsrc_t make_rsrc(const void *ptr, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)ptr, 0, bytes, 0x00020000);   // raw buffer, untyped dwords
}

// The wave's direct loads but the last N have landed and its own LDS reads are done, then the workgroup barrier.  Without the
// second wait the compiler leaves the reads of the tile just multiplied in flight across the barrier, and the loads requested
// behind it go into that tile's stage: an out-of-range one (zeros, no memory latency) can overtake them.
template <int N> __device__ __forceinline__ void wait_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

constexpr int NUM_XCD = 8;
constexpr uint32_t OOB = 0x80000000u;

// consecutive workgroup ids go to different XCDs; each XCD gets a contiguous run of the nblk tiles
__device__ __forceinline__ int xcd_run(int bid, int nblk)
{
    const int per = nblk / NUM_XCD, main = per * NUM_XCD;
    return bid < main ? (bid % NUM_XCD) * per + bid / NUM_XCD : bid;
}

}  // namespace

}  // namespace rl
