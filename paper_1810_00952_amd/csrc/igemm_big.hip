// Contraction at matrix-multiplication scale for gfx950, bf16 in / fp32 accumulate: 256 x 256 tiles of
//
//   C[m, n] = sum_k A[m, k] * Wp[n, k]          (a dense, or a 1x1 convolution at stride 1 of channel-last pixels)
//
// What bounds the 256 x 128 form of the pixel-on-lane kernel at these sizes is the operand bytes every workgroup requests and
// lets land in LDS (48 KB per 64 contraction indices and 2 Mi multiply-adds): without its direct loads a 256 x 256 kernel runs
// at the rate of its MFMAs alone (96 us for 4096^3, the library's 95), with them it does not.  A 256 x 256 tile moves a third
// less per MFMA, and wave tiles of 128 x 64 read six fragments for eight MFMAs instead of four for four.  Two stages of 64 KB:
// the barrier stands before the LAST of a tile's four k-steps, whose fragments are in registers by then, so that the tile after
// the next is requested into the stage being left (half between that step's MFMAs, half between the next's) and the next
// tile's first fragments are read under them.  Whole 128-byte lines per row: K tiles of 32 through four stages took 4 % longer,
// each line being fetched twice.  Four waves of 128 x 128 (fewer LDS reads, one wave per SIMD) 5 % longer.
// Measured: 4096^3 146 -> 122 us on one box, 118 -> 103 on another, 8192 x 4096 x 1024 78 -> 66 us, 4096 x 4096 x 512 25.6 -> 21.3 us.
// Eight waves (2 x 4), two per SIMD, 128 accumulator registers each.  Tile order, LDS swizzle, MFMA roles and the wave-private
// epilogue (64 rows at a time through the stages) as in igemm_lp.hip.
#include "igemm_lds.h"

namespace rl {

namespace {

template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

__device__ __forceinline__ void wg_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

}  // namespace

template <bool YF32>
__global__ __launch_bounds__(512) void igemm_big_kernel(const IgemmParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub; the body uses gfx950-only builtins
    constexpr int BKE = 64, BM = 256, BN = 256, WTM = 128, WTN = 64, TM = 4, TN = 2;
    constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
    constexpr int LPT = 8;                          // direct loads per wave and tile: four of A, four of W

    __shared__ __attribute__((aligned(1024))) unsigned char st0[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[STAGE];

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 2, wn = wave & 3;

    // each XCD a contiguous run of tiles; inside a run, channel tiles in groups of eight with the row tiles fastest
    const int nblk = p.nblk_m * p.nblk_n;
    int bid = blockIdx.x;
    {
        const int per = nblk / NUM_XCD, main = per * NUM_XCD;
        if (bid < main) bid = (bid % NUM_XCD) * per + bid / NUM_XCD;
    }
    int bm, bn;
    {
        constexpr int GN = 8;
        const int grp = bid / (GN * p.nblk_m);
        const int within = bid - grp * GN * p.nblk_m;
        const int gw = min(GN, p.nblk_n - grp * GN);
        bm = within / gw; bn = grp * GN + (within - bm * gw);
    }
    const int m0 = bm * BM, n0 = bn * BN;
    const rsrc_t rx = make_rsrc(p.x, p.x_bytes), rw = make_rsrc(p.w, p.w_bytes);

    // ---- requests: lane l of a load fills row l >> 3, position l & 7 of eight rows of 128 bytes
    uint32_t voff[LPT];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = (wave * 4 + i) * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row >> 1) & 7);
        const int m = m0 + row, n = min(n0 + row, p.N - 1);          // rows past N are computed on valid memory and never stored
        voff[i] = m < p.M ? (uint32_t)((int64_t)m * p.xs_w * 2) + chunk * 16 : OOB;
        voff[4 + i] = (uint32_t)((int64_t)n * p.Kp * 2) + chunk * 16;
    }
    const int nk = p.K / BKE;
    int f_kt = 0;
    uint32_t f_soff = 0;
    bool f_live = true;
#define RL_TILE_BEGIN { f_live = f_kt < nk; f_soff = f_live ? (uint32_t)f_kt * 128u : 0u; ++f_kt; }
#define RL_DMA(ST, D)                                                                                                 \
    __builtin_amdgcn_raw_ptr_buffer_load_lds((D) < 4 ? rx : rw, RL_LDS_PTR(ST + ((D) < 4 ? 0 : A_BYTES) + (wave * 4 + ((D) & 3)) * 1024), 16, \
                                             f_live ? voff[D] : OOB, f_soff, 0, 0);
#define RL_ISSUE(ST) { RL_TILE_BEGIN _Pragma("unroll") for (int d = 0; d < LPT; ++d) RL_DMA(ST, d) }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.0f;

    const int frow = lane & 31, fhalf = lane >> 5;
    int f_off[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) f_off[ks] = frow * 128 + (((2 * ks + fhalf) ^ ((frow >> 1) & 7)) << 4);
    u32x4 fw[2][TN], fx[2][TM];
#define RL_LOADP(ST, KS)                                                                                              \
    {                                                                                                                 \
        _Pragma("unroll") for (int j = 0; j < TN; ++j) fw[(KS) & 1][j] = *(const u32x4 *)(ST + A_BYTES + (wn * WTN + j * 32) * 128 + f_off[KS]); \
        _Pragma("unroll") for (int i = 0; i < TM; ++i) fx[(KS) & 1][i] = *(const u32x4 *)(ST + (wm * WTM + i * 32) * 128 + f_off[KS]);           \
        __builtin_amdgcn_sched_barrier(0);                                                                            \
    }
    // the eight MFMAs of a k-step; REQ 1, 2: direct loads 0-3, 4-7 of the tile being requested between them
#define RL_MMAP(KS, ISS, REQ)                                                                                         \
    {                                                                                                                 \
        _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                                \
            _Pragma("unroll") for (int j = 0; j < TN; ++j) {                                                          \
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fw[(KS) & 1][j]),      \
                                                                    __builtin_bit_cast(bf16x8, fx[(KS) & 1][i]), acc[i][j], 0, 0, 0); \
                if ((REQ) && (j & 1)) RL_DMA(ISS, 4 * (REQ) - 4 + i)                                                  \
                __builtin_amdgcn_sched_barrier(0);                                                                    \
            }                                                                                                         \
    }
    // Tile t in CUR, tile t+1 on its way into NXT.  The barrier stands before the LAST k-step of a tile: its fragments are in
    // registers, so that tile t+2 can be requested into CUR between its MFMAs, and tile t+1's first fragments are read there.
#define RL_BODY(CUR, NXT)                                          \
    {                                                              \
        RL_LOADP(CUR, 1)                                           \
        RL_MMAP(0, NXT, 2)                                         \
        RL_LOADP(CUR, 2)                                           \
        RL_MMAP(1, CUR, 0)                                         \
        RL_LOADP(CUR, 3)                                           \
        RL_MMAP(2, CUR, 0)                                         \
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); \
        RL_TILE_BEGIN                                              \
        RL_LOADP(NXT, 0)                                           \
        RL_MMAP(3, CUR, 1)                                         \
    }
    RL_ISSUE(st0)
    RL_TILE_BEGIN RL_DMA(st1, 0) RL_DMA(st1, 1) RL_DMA(st1, 2) RL_DMA(st1, 3)
    wait_vmcnt<4>();
    wg_barrier();
    RL_LOADP(st0, 0)
    int kt = 0;
#pragma unroll 1
    for (; kt + 2 <= nk; kt += 2) {
        RL_BODY(st0, st1)
        RL_BODY(st1, st0)
    }
    if (kt < nk) RL_BODY(st0, st1)
    wait_vmcnt<0>();             // the trailing out-of-range requests
#undef RL_BODY
#undef RL_MMAP
#undef RL_LOADP
#undef RL_ISSUE
#undef RL_DMA
#undef RL_TILE_BEGIN

    // ---- epilogue: from here each wave works alone in its own 16 KB of the stages, 64 of its 128 rows at a time
    wg_barrier();
    const Epilogue &e = p.epi;
    unsigned char *park = (wave < 4 ? st0 : st1) + (wave & 3) * 16384;
    const uint32_t y_bytes = p.y_bytes;
    const bool has_res = !YF32 && e.t_op >= 0;
    const rsrc_t rb = make_rsrc(e.has_bias ? e.bias_ptr : p.w, e.has_bias ? (uint32_t)p.N * 4u : 0u);     // absent: zeros without memory traffic
    const rsrc_t rres = make_rsrc(has_res ? e.t_ptr : p.w, has_res ? y_bytes : 0u);
    const rsrc_t ry = make_rsrc(p.y, y_bytes);
    const float lo = e.relu_last ? 0.0f : -INFINITY;
    f32x4 bias_r[TN][4];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int n = n0 + wn * WTN + 4 * fhalf + j * 32 + 8 * g;
            bias_r[j][g] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rb, n < p.N ? (uint32_t)n * 4u : OOB, 0, 0));
        }
    const int rr = lane >> 3, pp = lane & 7;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t y_off[8];
        u32x4 res_r[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int row = q * 8 + rr, cc = pp ^ ((row & 15) >> 1);
            const int m = m0 + wm * WTM + h * 64 + row, n = n0 + wn * WTN + cc * 8;
            y_off[q] = (m < p.M && n < p.N) ? (uint32_t)(((int64_t)m * p.ys_p + n) * (YF32 ? 4 : 2)) : OOB;
            if (!YF32) res_r[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rres, y_off[q], 0, 0));
        }
        if (h) wave_lds_exchange();          // the first half is read out
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int row = i * 32 + frow;
                    const int pos = (j * 8 + 2 * g + fhalf) ^ (row & 15);
                    f32x4 v;
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = acc[2 * h + i][j][4 * g + k] + bias_r[j][g][k];
                    *(f32x4 *)(park + row * 256 + pos * 16) = v;
                }
        wave_lds_exchange();
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int row = q * 8 + rr, pa = 2 * pp + (row & 1);
            const f32x4 a = *(const f32x4 *)(park + row * 256 + pa * 16);
            const f32x4 b = *(const f32x4 *)(park + row * 256 + (pa ^ 1) * 16);
            float v[8];
#pragma unroll
            for (int k = 0; k < 4; ++k) { v[k] = a[k]; v[4 + k] = b[k]; }
            if (YF32) {
                const u32x4 o0 = {__float_as_uint(fmaxf(v[0], lo)), __float_as_uint(fmaxf(v[1], lo)), __float_as_uint(fmaxf(v[2], lo)), __float_as_uint(fmaxf(v[3], lo))};
                const u32x4 o1 = {__float_as_uint(fmaxf(v[4], lo)), __float_as_uint(fmaxf(v[5], lo)), __float_as_uint(fmaxf(v[6], lo)), __float_as_uint(fmaxf(v[7], lo))};
                __builtin_amdgcn_raw_buffer_store_b128(o0, ry, y_off[q], 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(o1, ry, y_off[q] != OOB ? y_off[q] + 16u : OOB, 0, 0);
            } else {
                u32x4 o;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    v[2 * k] += __uint_as_float(res_r[q][k] << 16);
                    v[2 * k + 1] += __uint_as_float(res_r[q][k] & 0xffff0000u);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k] = pack_bf16x2(fmaxf(v[2 * k], lo), fmaxf(v[2 * k + 1], lo));
                __builtin_amdgcn_raw_buffer_store_b128(o, ry, y_off[q], 0, 0);
            }
        }
    }
#endif
}

template __global__ void igemm_big_kernel<false>(const IgemmParams);
template __global__ void igemm_big_kernel<true>(const IgemmParams);

// Rounds of workgroups times the time of one per 64 contraction indices: 1.9 us of a 256 x 256 tile against 1.14 of a 256 x 128 one
bool igemm_big_better(int64_t M, int64_t N, int64_t K)
{
    if (M < 256 || N < 256 || K % 64 != 0 || N % 8 != 0) return false;
    const int64_t big = ((M + 255) / 256) * ((N + 255) / 256), half = ((M + 255) / 256) * ((N + 127) / 128);
    return 1.9 * (double)((big + 255) / 256) < 1.14 * (double)((half + 255) / 256);
}

hipError_t launch_igemm_big(const IgemmParams &p0, hipStream_t s)
{
    IgemmParams p = p0;
    p.nblk_m = (p.M + 255) / 256;
    p.nblk_n = (p.N + 255) / 256;
    if (p.OHW == 1) p.xs_w = p.xs_n;             // elements from one row of A to the next: images of a dense, pixels of a convolution
    const int64_t nblk = (int64_t)p.nblk_m * p.nblk_n;
    // rows of whole 16-byte chunks one after the other, whole K tiles, [f32 bias] [+ bf16 residual] [relu]
    if (p.in_dtype != DT_BF16 || p.x2 || p.KH * p.KW != 1 || p.sh != 1 || p.sw != 1 || p.ph || p.pw || p.K % 64 != 0 || p.K < 64 || p.K1 != p.K || p.xs_w % 8 || p.Kp % 8 ||
        p.N % 8 || p.ys_c != 1 || p.ys_n != (int64_t)p.OHW * p.ys_p || p.ys_p % 8 || (p.epi.rest_n > 0 && !p.epi.relu_last) ||
        (p.epi.t_op >= 0 && (p.epi.t_op != E_ADD || p.epi.t_dtype != DT_BF16 || p.y_dtype != DT_BF16)) || nblk <= 0 || nblk > 0x7fffffff ||
        ((uint64_t)(p.M - 1) * p.xs_w + p.K) * 2 > p.x_bytes || ((uint64_t)(p.N - 1) * p.Kp + p.K) * 2 > p.w_bytes)
        return hipErrorInvalidValue;
    if (p.y_dtype == DT_BF16) hipLaunchKernelGGL(igemm_big_kernel<false>, dim3((unsigned)nblk), dim3(512), 0, s, p);
    else hipLaunchKernelGGL(igemm_big_kernel<true>, dim3((unsigned)nblk), dim3(512), 0, s, p);
    return hipGetLastError();
}

}  // namespace rl
