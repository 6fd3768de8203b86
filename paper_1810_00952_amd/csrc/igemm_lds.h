// What the contraction kernels share: descriptors, direct global -> LDS loads, the K loop's barrier, the order of the XCDs.
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

// the same for loads written out below
__device__ __forceinline__ u32x4 make_desc(const void *ptr, uint32_t bytes)
{
    const uint64_t a = (uint64_t)ptr;
    u32x4 d = {(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, bytes, 0x00020000u};
    return d;
}

// One direct load: 64 lanes x 16 bytes from desc[voff + soff] to LDS at lds_addr + lane*16.  Written out because the compiler would make
// every read of the stages wait for all requests into them; where it is used they are counted by hand.
__device__ __forceinline__ void dma16(const u32x4 &desc, uint32_t lds_addr, uint32_t voff, uint32_t soff)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds_addr), "v"(voff), "s"(desc), "s"(soff) : "memory");
#endif
}
__device__ __forceinline__ void dma16(const u32x4 &desc, uint32_t lds_addr, uint32_t voff)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(lds_addr), "v"(voff), "s"(desc) : "memory");
#endif
}

// The wave's direct loads but the last N have landed and its own LDS reads are done, then the workgroup barrier.  Without the
// second wait the compiler leaves the reads of the tile just multiplied in flight across the barrier, and the loads requested
// behind it go into that tile's stage: an out-of-range one (zeros, no memory latency) can overtake them.
template <int N> __device__ __forceinline__ void wait_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

constexpr int NUM_XCD = 8;
constexpr uint32_t OOB = 0x80000000u;       // past every descriptor's extent (below 2^31): reads as zero, no memory traffic

// elements of a 16-byte vector
template <typename T> struct Elem;
template <> struct Elem<float> { static constexpr int KV = 4; };
template <> struct Elem<uint16_t> { static constexpr int KV = 8; };

// consecutive workgroup ids go to different XCDs; each XCD gets a contiguous run of the nblk tiles
__device__ __forceinline__ int xcd_run(int bid, int nblk)
{
    const int per = nblk / NUM_XCD, main = per * NUM_XCD;
    return bid < main ? (bid % NUM_XCD) * per + bid / NUM_XCD : bid;
}

}  // namespace

}  // namespace rl
