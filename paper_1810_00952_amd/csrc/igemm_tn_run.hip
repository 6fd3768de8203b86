// The contraction over rows (igemm_tn.hip) of a 3x3, stride 1, pad 1 weight gradient in bf16: the three taps of a filter row from one
// copy of the rows.
//
// What bounds the general form is LDS: a 64x64 tile of one tap fills 16 KB and reads 32 KB for 16 MFMAs, 384 cycles of LDS for 128 of
// MFMA.  At stride 1 on an unchanged image size tap (kh, kw) of flat pixel p (over all images) is flat input pixel
// p + (kh - 1) W + kw - 1, so the taps kw = 0, 1, 2 of one kh read the same rows of x, a row apart.  A workgroup has 64 output channels,
// 64 input channels and the three taps of one kh: 16 KB filled and 40 KB read for 48 MFMAs, 450 cycles of LDS for 384 of MFMA.
//   * x rows lie in a ring of eight stages of 64 pixels, shifted by one: stage u holds the rows of centre pixels 64 u - 1 .. 64 u + 62, so
//     that a K tile of 64 pixels reads its stage and the first two rows of the next.  A row whose kh lies outside its image arrives as
//     zeros (an out-of-range request).  Where kw leaves the image row, and past the last pixel, the lane's transposing read is aimed
//     at zeros: nothing that does not belong there is ever multiplied, not even by a zero.
//   * Eight waves: two halves of the input channels x four quarters of each K tile (16 pixels), a wave's 64 x 32 x 3 taps from five
//     fragments for six MFMAs.  The fragments of tile u + 1 are read between the MFMAs of tile u, and the stage that tile u has left is
//     requested again behind the barrier that follows: five K tiles of requests in flight.
//   * The quarters' sums meet in LDS at the end, ((q0 + q1) + (q2 + q3)); slices of K and their adding launch as in igemm_tn.hip.
// Measured, 64x128x28x28 -> 128 in bf16, 21 slices: 30.6 -> 24.6 us (600 TFLOP/s; both gradients of the layer 73.7 -> 70.4).  A K tile takes
// about 600 cycles, and 12 us go into start, end and the sums' way to memory, which is why short slices stay with the square tiles
// (Planner::run_weight_gradients).  Layers, before and after: 64x256x14x14 -> 256 71.9 -> 67.6, 48x200x20x23 -> 136 95.5 -> 82.6,
// 20x256x28x28 -> 256 78.8 -> 71.8, 64x64x56x56 -> 64 99.7 -> 95.2, 64x512x7x7 -> 512 60.7 -> 57.7.
// The swizzle is that of igemm_tn.h: rows r and r + 2 differ in it for odd r as well, so a shift by a row costs no bank conflict.
#include <algorithm>

#include "igemm_lds.h"

namespace rl {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int NB = 8;                             // stages, a power of two
constexpr int ST = 64 * 128;                      // bytes per stage of either operand: 64 rows of 64 channels
constexpr int RING = NB * ST, A_OFF = RING, Z_OFF = 2 * RING, LDS_BYTES = Z_OFF + 256;
static_assert(4 * 96 * 64 * 4 <= Z_OFF && LDS_BYTES <= 160 * 1024, "LDS holds the sums of four waves");

__device__ __forceinline__ int key(int row) { return ((row >> 1) & 1) << 2; }      // in 16-byte chunks of a row of eight

}  // namespace

__global__ __launch_bounds__(512) void igemm_tn_run_kernel(const TnParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub; the body uses gfx950-only builtins
    __shared__ __attribute__((aligned(1024))) unsigned char lds[LDS_BYTES];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wn = wave & 1, kq = wave >> 1;
    const uint32_t lds_a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)lds;

    // workgroups of one slice share its rows: slices in order, each XCD a contiguous run
    const int tiles = p.nblk_m * p.nblk_n;
    const int bid = xcd_run(blockIdx.x, tiles * p.splits);
    const int split = bid / tiles, tile = bid - split * tiles;
    const int bm = tile / p.nblk_n, bn = tile - bm * p.nblk_n;     // bn: (block of input channels, kh)
    const int kh = bn % 3, m0 = bm * 64, c0 = bn / 3 * 64;
    const int W = p.W, P = p.P;
    const int kt0 = split * p.split_tiles, nk = min((P + 63) / 64 - kt0, p.split_tiles);      // K tiles of the slice

    if (t < 64) ((uint32_t *)(lds + Z_OFF))[t] = 0u;

    // ---- requests: one of A and one of x per wave and K tile, eight rows each.  Everything that changes from tile to tile is carried
    // along (a division per row costs more than the tile's MFMAs): offsets, and line and column of x's centre pixel.  Rows past
    // the slice lie outside the descriptors, but for the row after it that its last pixel's kw = 2 reads
    const int row = wave * 8 + (lane >> 3);
    const int col = ((lane & 7) ^ key(row)) * 8;
    const uint32_t lda = (uint32_t)p.lda * 2, ldb = (uint32_t)p.ldb * 2;
    const int end = min(P, (kt0 + nk) * 64);
    const u32x4 da = make_desc(p.a, (uint32_t)end * lda), dx = make_desc(p.b, (uint32_t)min(P, max(0, end + 1 + (kh - 1) * W)) * ldb);
    auto div = [](int n, int d, uint32_t mul, uint32_t sh) { return d == 1 ? n : (int)(__umulhi((uint32_t)n, mul) >> sh); };
    const int f0 = kt0 * 64 + row - 1;                // the first tile's centre pixel of x
    uint32_t off_a = m0 + col < p.M ? (uint32_t)(f0 + 1) * lda + (uint32_t)(m0 + col) * 2 : OOB;
    uint32_t off_x = c0 + col < p.C ? (uint32_t)(f0 + (kh - 1) * W) * ldb + (uint32_t)(c0 + col) * 2 : OOB;
    const int line0 = div(f0 + p.OHW, p.OW, p.div_ow_mul, p.div_ow_sh);      // (one image ahead: the first pixel's is -1)
    uint32_t x_ow = (uint32_t)(f0 + p.OHW - line0 * W), x_oh = (uint32_t)(line0 - div(f0 + p.OHW, p.OHW, p.div_ohw_mul, p.div_ohw_sh) * p.H);
    const uint32_t d_ow = 64 % W, d_oh = 64 / W % p.H, step_a = 64 * lda, step_x = 64 * ldb;
    const uint32_t outside = kh == 0 ? 0u : kh == 2 ? (uint32_t)p.H - 1 : ~0u;      // the line whose row kh lies outside the image
    auto issue = [&](int stage) {                     // the next K tile; pixels past the last go on as another image's
        const uint32_t at = lds_a + (uint32_t)(stage + wave * 1024);
        dma16(da, at + A_OFF, off_a);
        dma16(dx, at, x_oh == outside ? OOB : off_x);
        off_a += step_a;
        off_x += step_x;
        x_ow += d_ow;
        x_oh += d_oh + (x_ow >= (uint32_t)W ? 1u : 0u);
        x_ow = min(x_ow, x_ow - (uint32_t)W);
        x_oh = min(x_oh, x_oh - (uint32_t)p.H);
    };

    // ---- fragments: lane q of a group of sixteen reads row q / 4 of the group's 4 x 16 block, columns 4 (q & 3) ..
    const int g4 = lane >> 4, q = lane & 15;
    const int kr = kq * 16 + (g4 >> 1) * 8 + (q >> 2), cc = (g4 & 1) * 2 + ((q & 3) >> 1), half = (q & 1) * 8;
    int fa[2], fx[3];
#pragma unroll
    for (int i = 0; i < 2; ++i) fa[i] = kr * 128 + (((i * 4 + cc) ^ key(kr)) << 4) + half;
#pragma unroll
    for (int k = 0; k < 3; ++k) fx[k] = (kr + k) * 128 + (((wn * 4 + cc) ^ key(kr + k)) << 4) + half;
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    auto tr4 = [&](int off) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(lds + off)); };

    s16x4 ra[2][2][2], rx[2][3][2];                   // [set][tile or tap][four pixels]
    f32x16 acc[2][3];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][k][e] = 0.0f;

    // lines' ends: column of the lane's pixels in the tile whose fragments are read next.  (Pixels past the last: their rows of x are
    // zeros, but for the one before the first of them, and that one starts a line.)
    uint32_t ow[2];
    int at_x[3][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int px = kt0 * 64 + kr + 4 * h;
        ow[h] = (uint32_t)(px - div(px, p.OW, p.div_ow_mul, p.div_ow_sh) * W);
    }
    int at_a[2];
    auto aim = [&](int stage) {
        at_a[0] = A_OFF + stage + fa[0];
        at_a[1] = A_OFF + stage + fa[1];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int in = (stage + fx[k] + 512 * h) & (RING - 1);
                at_x[k][h] = (k == 0 && ow[h] == 0u) || (k == 2 && ow[h] == (uint32_t)W - 1) ? Z_OFF + half : in;
            }
            ow[h] += d_ow;
            ow[h] = min(ow[h], ow[h] - (uint32_t)W);
        }
    };
    auto read = [&](int set, int i) {                 // read i of ten
        if (i < 4) ra[set][i >> 1][i & 1] = tr4(at_a[i >> 1] + 512 * (i & 1));
        else rx[set][(i - 4) >> 1][i & 1] = tr4(at_x[(i - 4) >> 1][i & 1]);
    };
    auto frag = [](const s16x4 &lo, const s16x4 &hi) { return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)); };

#pragma unroll 1
    for (int u = 0; u < NB; ++u) issue(u * ST);
    wait_barrier<2 * (NB - 2)>();                     // tiles 0 and 1 are there
    aim(0);
#pragma unroll
    for (int i = 0; i < 10; ++i) read(0, i);
    // On entry of a tile, u: its fragments (register set u % 2) are read or on their way, requests are out up to tile u + NB - 1.  The
    // wait leaves all but those of tiles u + 3 .. behind, and this wave's own reads; the barrier says so for all waves: tile u's
    // stage of either operand has no reader left
    int stage = 0;
    auto multiply = [&](int set) {
        wait_barrier<2 * (NB - 3)>();
        issue(stage);
        stage = (stage + ST) & (RING - 1);
        aim(stage);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                acc[i][k] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(ra[set][i][0], ra[set][i][1]), frag(rx[set][k][0], rx[set][k][1]), acc[i][k], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (2 * k + i < 5) {
                    read(set ^ 1, 2 * (2 * k + i));
                    read(set ^ 1, 2 * (2 * k + i) + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    // (eight tiles a trip, the stages constants, took 25.5 us where two took 26.8, both with the end below unrolled: 40 KB of code.  Two
    // with it rolled, 6 KB: 24.6)
    int left = nk;
#pragma unroll 1
    for (;;) {
        multiply(0);
        if (--left == 0) break;
        multiply(1);
        if (--left == 0) break;
    }
    wait_barrier<0>();                                // the trailing requests, too

    // ---- the quarters' sums: 1 and 3 hand theirs to 0 and 2, whose sums all threads then add and store, four rows of a column at a
    // time.  (Rolled, as the K loop is: a workgroup meets its code cold.)
    // register 4g + e of lane l holds row 8g + 4 (l >> 5) + e, column l & 31 of its 32 x 32 tile
    f32x4 *park = (f32x4 *)lds;
    const int place = (((kq >> 1) * 2 + wn) * 24) * 64 + lane;
    auto put = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    park[place + (i * 12 + k * 4 + g) * 64] = f32x4{acc[i][k][4 * g], acc[i][k][4 * g + 1], acc[i][k][4 * g + 2], acc[i][k][4 * g + 3]};
    };
    if (kq & 1) put();
    __syncthreads();
    if (!(kq & 1)) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 v = park[place + (i * 12 + k * 4 + g) * 64];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][k][4 * g + e] += v[e];
                }
        put();
    }
    __syncthreads();
#pragma unroll 1
    for (int j = 0; j < 6; ++j) {
        const int grp = wave + 8 * j;                  // (half of the input channels, tile of output channels, tap, group of registers)
        const f32x4 v0 = park[grp * 64 + lane], v1 = park[(48 + grp) * 64 + lane];
        const int i = grp / 12 & 1, kw = grp / 4 % 3, c = c0 + grp / 24 * 32 + (lane & 31);
        const int m = m0 + i * 32 + 8 * (grp & 3) + 4 * (lane >> 5), tap = kh * 3 + kw;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float v = v0[e] + v1[e];
            if (c >= p.C || m + e >= p.M) continue;
            if (p.splits > 1) p.partial[((int64_t)split * p.M + m + e) * p.N + tap * p.C + c] = v;
            else if (c < p.Cout && m + e < p.Mout) store_from_f32(p.y, p.y_dtype, ((int64_t)(m + e) * p.Cout + c) * p.T + tap, v);
        }
    }
#endif
}

bool igemm_tn_run_ok(const TnParams &p, int32_t dtype)
{
    return dtype == DT_BF16 && p.conv && p.T == 9 && p.KW == 3 && p.s == 1 && p.ph == 1 && p.pw == 1 && p.OW == p.W && p.OHW == p.H * p.W && p.lda < 65536 && p.ldb < 65536;     // (offsets a few hundred rows past the last don't wrap)
}

bool igemm_tn_prepare(TnParams &p, int element_size, int tile);                 // igemm_tn.hip
hipError_t launch_tn_reduce(const TnParams &p, hipStream_t s);

hipError_t launch_igemm_tn_run(const TnParams &p0, int32_t dtype, hipStream_t s)
{
    TnParams p = p0;
    if (!igemm_tn_run_ok(p, dtype) || !igemm_tn_prepare(p, 2, 64) || p.P % p.OHW != 0) return hipErrorInvalidValue;
    p.nblk_n = (p.C + 63) / 64 * 3;
    const int64_t grid = (int64_t)p.nblk_m * p.nblk_n * p.splits;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(igemm_tn_run_kernel, dim3((unsigned)grid), dim3(512), 0, s, p);
    const hipError_t er = hipGetLastError();
    return er != hipSuccess || p.splits == 1 ? er : launch_tn_reduce(p, s);
}

}  // namespace rl
