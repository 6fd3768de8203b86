// Implicit-GEMM contraction for gfx950, LDS-DMA variant: operand tiles go
// from global memory straight into LDS (buffer_load ... lds, 16 bytes per
// lane), three K tiles deep, with no staging registers and no LDS stores in
// the K loop.
//
//   C[m, n] = sum_k A[m, k] * Wp[n, k],  m = (image, oh, ow), n = out channel,
//   k = (kh, kw, c)
//
// Preconditions (checked by the planner): channel-last activations with
// C a multiple of the K tile (64 bf16 / 32 f32), so a K tile lies inside one
// filter tap and the tap state is wave-uniform; K a multiple of the tile and at
// least two tiles; KH*KW <= 32; operands below 2 GiB.
//
// Tile layout in LDS: rows of 128 bytes (8 chunks of 16 bytes), unpadded,
// because one DMA instruction writes 64 lanes x 16 bytes contiguously = 8 rows.
// Bank conflicts are avoided by choosing which global chunk each lane fetches:
// position p of row r holds chunk p ^ ((r >> 1) & 7), so the 16 rows read by a
// quarter-wave fragment load cover all 64 banks once.
//
// TAPS form: channel counts that are a multiple of the 16-byte vector only.  A K tile then spans filter taps; every lane
// decodes, per K tile, the tap and channel of its own 16-byte chunk (two chunks per lane: the swizzle key alternates with the
// row group) by multiply-high, and its rows' taps are checked against the image one by one.  What it replaces staged the
// same tiles through registers: 17x96x29x29 -> 136 3x3 bf16 with residual, contraction alone 58 us against 15.
//
// STORE_ANY form: results in Shape order (channel-first) or with ragged N, kept apart from the row-wise form so that neither
// pays for the other's registers and code.
//
// Padding taps and rows past M get a buffer offset outside the descriptor's
// range: the hardware then writes zeros into LDS without touching memory.
//
// Synchronisation: each stage is its own LDS array so that the compiler's
// wait-count insertion can tell DMA writes to one stage from fragment reads of
// another; the waits on the DMA itself are explicit (s_waitcnt vmcnt) and the
// workgroup barrier is the bare instruction, one per K tile:
//     wait(my DMAs of tile t) ; barrier ; issue DMA of tile t+2 ; MFMAs on tile t
// After the barrier every wave's part of tile t has landed and every wave has
// left tile t-1, whose stage the new DMA overwrites.
#include <algorithm>

#include "igemm_dma.h"

namespace rl {

// The second kernel of a split contraction: y[m, n] = epilogue(partial[0][m][n] + partial[1][m][n] + ...), one element
// per thread, slices added in order (so the result does not depend on timing), any output strides.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const IgemmParams p)
{
    touch_args(p);
    const Epilogue &e = p.epi;
    const uint32_t total = (uint32_t)p.M * (uint32_t)p.N;            // below 2^31 (checked by the launcher): 32-bit index arithmetic
    for (uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += gridDim.x * blockDim.x) {
        const int m = (int)(idx / (uint32_t)p.N), n = (int)(idx - (uint32_t)m * (uint32_t)p.N);
        // eight slices' values are requested before the first is added (the additions stay in slice order)
        float val = 0.0f;
        for (int z0 = 0; z0 < p.splits; z0 += 8) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = z0 + j < p.splits ? p.partial[(int64_t)(z0 + j) * total + idx] : 0.0f;    // splits * total < 2^26 floats
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (z0 + j < p.splits) val = z0 + j == 0 ? v[j] : val + v[j];
        }
        const int img = m / p.OHW, pix = m - img * p.OHW;
        const int64_t off = (int64_t)img * p.ys_n + (int64_t)pix * p.ys_p + (int64_t)n * p.ys_c;
        for (int s = 0; s < e.n_ops; ++s) val = epi_step(e, s, val, off, n);
        store_from_f32(p.y, p.y_dtype, off, val);
    }
}

hipError_t launch_splitk_reduce(const IgemmParams &p, hipStream_t s)
{
    const int64_t total = (int64_t)p.M * p.N;
    if (total < 1 || total * p.splits >= (int64_t)1 << 31 || !p.partial) return hipErrorInvalidValue;
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)std::min<int64_t>((total + 255) / 256, 256 * 16)), dim3(256), 0, s, p);
    return hipGetLastError();
}

// The adding launch of a split dense contraction together with the small dense layer that consumes its result: one
// workgroup per row.  Threads add the slices of their columns in slice order and apply the first group's epilogue
// (and the rounding to the dtype the tensor between the groups has), the row meets in LDS, then every wave takes
// output columns in turn: lanes multiply a strided share of the row, the 64 shares are added in a fixed tree.
// A chain of memory latencies and nothing else, so everything whose address is known is requested at the start: the slices, both
// biases and the weights of a wave's first JP outputs (NI: shares of a row per lane).  32 rows, 128 -> 10: 6.1 us by the trace -> 5.4; 64 rows,
// 500 -> 10: 9.6 -> 6.2 (one output of a wave after the other, its weights behind the barrier, on 256 threads).
constexpr int ADD_WAVES = 8;
template <int NI, int JP>
__global__ __launch_bounds__(64 * ADD_WAVES) void reduce_dense_kernel(const ReduceDenseParams p)
{
    __shared__ float hs[64 * NI];
    touch_args(p);
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int m = blockIdx.x;
    const int64_t slice = (int64_t)p.M * p.N1;
    auto weight = [&](int j, int i) -> float {
        const int n = lane + 64 * i;
        return j < p.N2 && n < p.N1 ? load_as_f32(p.w2, p.w_dtype, (int64_t)j * p.Kp2 + n) : 0.0f;
    };
    const bool early = NI <= 8;
    float w[JP][NI <= 8 ? NI : 1], b2[JP];
#pragma unroll
    for (int q = 0; q < JP; ++q) {
        const int j = wave + ADD_WAVES * q;
        b2[q] = p.epi2.simple && p.epi2.has_bias && j < p.N2 ? load_as_f32(p.epi2.bias_ptr, p.epi2.bias_dtype, j) : 0.0f;
        if constexpr (NI <= 8) {
#pragma unroll
            for (int i = 0; i < NI; ++i) w[q][i] = weight(j, i);
        }
    }
    for (int n = t; n < p.N1; n += 64 * ADD_WAVES) {
        const float *src = p.partial + (int64_t)m * p.N1 + n;
        const float b1 = p.epi1.simple && p.epi1.has_bias ? load_as_f32(p.epi1.bias_ptr, p.epi1.bias_dtype, n) : 0.0f;
        float val = 0.0f;
        for (int z0 = 0; z0 < p.splits; z0 += 16) {
            float v[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = z0 + j < p.splits ? src[(int64_t)(z0 + j) * slice] : 0.0f;
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (z0 + j < p.splits) val = z0 + j == 0 ? v[j] : val + v[j];
        }
        const int64_t off = (int64_t)m * p.hs_n + (int64_t)n * p.hs_c;
        if (p.epi1.simple && p.epi1.t_op < 0) {
            val += b1;
            uint64_t codes = p.epi1.rest_ops;
            for (int s = 0; s < p.epi1.rest_n; ++s, codes >>= 8) val = unary_step((int)(codes & 0xff), val);
        } else {
            for (int s = 0; s < p.epi1.n_ops; ++s) val = epi_step(p.epi1, s, val, off, n);
        }
        hs[n] = p.h_dtype == DT_BF16 ? round_bf16(val) : val;
    }
    __syncthreads();
    for (int j0 = wave; j0 < p.N2; j0 += ADD_WAVES * JP) {
        float acc[JP];
#pragma unroll
        for (int q = 0; q < JP; ++q) {
            acc[q] = 0.0f;
            if constexpr (NI <= 8) {
                if (j0 != wave) {
#pragma unroll
                    for (int i = 0; i < NI; ++i) w[q][i] = weight(j0 + ADD_WAVES * q, i);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < JP; ++q) {
            if constexpr (NI <= 8) {
#pragma unroll
                for (int i = 0; i < NI; ++i)
                    if (lane + 64 * i < p.N1) acc[q] += hs[lane + 64 * i] * w[q][i];
            } else if (j0 + ADD_WAVES * q < p.N2) {
                for (int n = lane; n < p.N1; n += 64) acc[q] += hs[n] * load_as_f32(p.w2, p.w_dtype, (int64_t)(j0 + ADD_WAVES * q) * p.Kp2 + n);
            }
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
            for (int q = 0; q < JP; ++q) acc[q] += __shfl_xor(acc[q], d, 64);
#pragma unroll
        for (int q = 0; q < JP; ++q) {
            const int j = j0 + ADD_WAVES * q;
            if (lane != q || j >= p.N2) continue;
            const int64_t off = (int64_t)m * p.ys_n + (int64_t)j * p.ys_c;
            float v = acc[q];
            if (p.epi2.simple && p.epi2.t_op < 0 && early) {
                v += j0 == wave ? b2[q] : p.epi2.has_bias ? load_as_f32(p.epi2.bias_ptr, p.epi2.bias_dtype, j) : 0.0f;
                uint64_t codes = p.epi2.rest_ops;
                for (int s = 0; s < p.epi2.rest_n; ++s, codes >>= 8) v = unary_step((int)(codes & 0xff), v);
            } else {
                for (int s = 0; s < p.epi2.n_ops; ++s) v = epi_step(p.epi2, s, v, off, j);
            }
            store_from_f32(p.y, p.y_dtype, off, v);
        }
    }
}

hipError_t launch_reduce_dense(const ReduceDenseParams &p, hipStream_t s)
{
    if (!p.partial || !p.w2 || !p.y || p.splits < 2 || p.splits > 64 || p.M < 1 || p.M > 65535 || p.N1 < 1 || p.N1 > REDUCE_DENSE_MAX_N1 ||
        p.N2 < 1 || p.N2 > REDUCE_DENSE_MAX_N2 || p.Kp2 < p.N1 || (int64_t)p.M * p.N1 * p.splits >= (int64_t)1 << 31)
        return hipErrorInvalidValue;
#define RL_GO(NI, JP) hipLaunchKernelGGL((reduce_dense_kernel<NI, JP>), dim3((unsigned)p.M), dim3(64 * ADD_WAVES), 0, s, p)
    // up to an output a wave: nothing is asked for ahead that is not there, and the row's shares fit closer (99 rows, 768 -> 128 -> 4 f32
    // 10.7 us the two layers, now 9.9, 768 -> 256 -> 8 11.15 and 10.4; from 9 outputs on the other form, 768 -> 128 -> 24 11.4)
    if (p.N2 <= 8) {
        if (p.N1 <= 128) RL_GO(2, 1);
        else if (p.N1 <= 256) RL_GO(4, 1);
        else if (p.N1 <= 512) RL_GO(8, 1);
        else RL_GO(REDUCE_DENSE_MAX_N1 / 64, 1);
    } else if (p.N1 <= 128) RL_GO(2, 4);
    else if (p.N1 <= 512) RL_GO(8, 2);
    else RL_GO(REDUCE_DENSE_MAX_N1 / 64, 2);
#undef RL_GO
    return hipGetLastError();
}

// explicit instantiations (the host-side launch stubs of a kernel template with function-local
// __shared__ arrays are not emitted implicitly)
#define RL_ONE(T, BM, BN, MODE, TAPS, TEAMS) template __global__ void igemm_dma_kernel<T, BM, BN, MODE, TAPS, Alone, TEAMS>(const IgemmParams, const Alone);
#define RL_INST(T, BM, BN, MODE, TAPS) RL_ONE(T, BM, BN, MODE, TAPS, 1)
#define RL_TWO(T) RL_ONE(T, 64, 64, STORE_ROWS, false, 2) RL_ONE(T, 64, 64, STORE_ANY, false, 2) RL_ONE(T, 64, 64, STORE_ROWS, true, 2) RL_ONE(T, 64, 64, STORE_ANY, true, 2)
RL_TWO(uint16_t) RL_TWO(float)
#undef RL_TWO
#define RL_INST4(T, BM, BN) RL_INST(T, BM, BN, STORE_ROWS, false) RL_INST(T, BM, BN, STORE_ANY, false) RL_INST(T, BM, BN, STORE_ROWS, true) RL_INST(T, BM, BN, STORE_ANY, true)
RL_INST(uint16_t, 128, 128, STORE_ROWS, false) RL_INST(uint16_t, 128, 128, STORE_ANY, false) RL_INST4(uint16_t, 128, 64) RL_INST4(uint16_t, 64, 64) RL_INST(uint16_t, 64, 64, STORE_GATES, false)
RL_INST4(float, 128, 64) RL_INST4(float, 64, 64) RL_INST(float, 64, 64, STORE_GATES, false)
#undef RL_INST4
#undef RL_INST
#undef RL_ONE
#define RL_INST(NI, JP) template __global__ void reduce_dense_kernel<NI, JP>(const ReduceDenseParams);
RL_INST(2, 4) RL_INST(8, 2) RL_INST(REDUCE_DENSE_MAX_N1 / 64, 2)
RL_INST(2, 1) RL_INST(4, 1) RL_INST(8, 1) RL_INST(REDUCE_DENSE_MAX_N1 / 64, 1)
#undef RL_INST

// what the kernel's K loop assumes of the operands
bool igemm_dma_takes(const IgemmParams &p, bool taps, int element_size)
{
    // chunks of one tap and channel run, no concatenation
    if (taps) return p.C % (16 / element_size) == 0 && p.K == p.C * p.KH * p.KW && p.K1 == p.K && !p.x2 && p.Kp >= p.K;
    // a partial last K tile: one tap, no concatenation, weight rows padded to whole tiles
    const int BKE = 128 / element_size;
    return p.K % BKE == 0 || (p.KH * p.KW == 1 && p.K1 == p.K && !p.x2 && p.Kp % BKE == 0 && p.Kp >= p.K);
}

// every slice holds at least one K tile and the slices cover K exactly once
bool igemm_dma_splits_ok(const IgemmParams &p, bool taps, int element_size)
{
    const int BKE = 128 / element_size, nk = (p.K + BKE - 1) / BKE;
    return p.partial && p.splits <= 64 && (int64_t)p.M * p.N * p.splits < (int64_t)1 << 31 && p.split_tiles >= 1 && (int64_t)(p.splits - 1) * p.split_tiles < nk &&
           (int64_t)p.splits * p.split_tiles >= nk && (taps || p.C % BKE == 0 || p.KH * p.KW == 1) && p.K1 == p.K;
}

template <typename T, int BM, int BN, bool GATES, bool TAPS, int TEAMS>
static void go_dma(const IgemmParams &p, unsigned nblk, hipStream_t s)
{
    const bool rows = p.splits > 1 || (p.ys_n == (int64_t)p.OHW * p.ys_p && p.ys_c == 1 && (p.N & 7) == 0 && (p.ys_p & 7) == 0);
    const dim3 grid(nblk, (unsigned)std::max(p.splits, 1));
    if constexpr (GATES) hipLaunchKernelGGL((igemm_dma_kernel<T, 64, 64, STORE_GATES, false, Alone, 1>), grid, dim3(256), 0, s, p, Alone{});
    else if (rows) hipLaunchKernelGGL((igemm_dma_kernel<T, BM, BN, STORE_ROWS, TAPS, Alone, TEAMS>), grid, dim3(256 * TEAMS), 0, s, p, Alone{});
    else hipLaunchKernelGGL((igemm_dma_kernel<T, BM, BN, STORE_ANY, TAPS, Alone, TEAMS>), grid, dim3(256 * TEAMS), 0, s, p, Alone{});
}

template <typename T, int BM, int BN, bool GATES, bool TAPS>
static hipError_t launch_dma(const IgemmParams &p0, hipStream_t s)
{
    IgemmParams p = p0;
    if (!igemm_dma_takes(p, TAPS, (int)sizeof(T)) || (GATES && (TAPS || p.K % (128 / (int)sizeof(T)) != 0))) return hipErrorInvalidValue;
    p.nblk_m = (p.M + BM - 1) / BM;
    p.nblk_n = (p.N + BN - 1) / BN;
    int64_t nblk = (int64_t)p.nblk_m * p.nblk_n;
    if (nblk <= 0 || nblk > 0x7fffffff) return hipErrorInvalidValue;
    if (p.splits > 1 && (GATES || !igemm_dma_splits_ok(p, TAPS, (int)sizeof(T)))) return hipErrorInvalidValue;
    if constexpr (BM == 64 && BN == 64 && !GATES) {
        if (p.splits <= 1 && nblk <= 256) go_dma<T, 64, 64, false, TAPS, 2>(p, (unsigned)nblk, s);
        else go_dma<T, 64, 64, false, TAPS, 1>(p, (unsigned)nblk, s);
    } else go_dma<T, BM, BN, GATES, TAPS, 1>(p, (unsigned)nblk, s);
    hipError_t er = hipGetLastError();
    if (er != hipSuccess || p.splits <= 1 || p.skip_reduce) return er;
    return launch_splitk_reduce(p, s);
}

template <typename T, bool TAPS>
static hipError_t launch_dma_typed(const IgemmParams &p, const IgemmLaunch &l, hipStream_t s)
{
    if (l.gates) {
        if (l.tile != TILE_64x64 || TAPS) return hipErrorInvalidValue;
        return launch_dma<T, 64, 64, true, false>(p, s);
    }
    switch (l.tile) {
    case TILE_128x128:                     // bf16 within a tap only: the planner takes smaller tiles for everything else
        if constexpr (TAPS || sizeof(T) == 4) return hipErrorInvalidValue;
        else return launch_dma<T, 128, 128, false, false>(p, s);
    case TILE_128x64: return launch_dma<T, 128, 64, false, TAPS>(p, s);
    default: return launch_dma<T, 64, 64, false, TAPS>(p, s);
    }
}

hipError_t launch_igemm_dma(const IgemmParams &p, const IgemmLaunch &l, hipStream_t s)
{
    if (p.in_dtype == DT_BF16) return l.taps ? launch_dma_typed<uint16_t, true>(p, l, s) : launch_dma_typed<uint16_t, false>(p, l, s);
    return l.taps ? launch_dma_typed<float, true>(p, l, s) : launch_dma_typed<float, false>(p, l, s);
}

}  // namespace rl
