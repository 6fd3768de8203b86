// Contraction over the SLOW axis of both operands:
//
//   C[m, j] = sum_p A[p, m] * B[row(p, tap), c],   j = (tap, c), tap = (kh, kw)
//
// the form of every weight gradient: A = dy with its channels fastest ([pixel][O], or [batch row][feature] of a dense),
// B = x with its channels fastest ([image][H][W][C]); p runs over the output pixels of the whole batch, and tap (kh, kw)
// of output pixel (n, oh, ow) is row (n, oh s - ph + kh, ow s - pw + kw) of x, or nothing outside the image.  A dense, and
// a 1x1 convolution at stride 1 without padding, have row(p) = p.
//
// What bounds it: an MFMA wants consecutive contraction indices per lane, and here they are a row apart.  bf16: K tiles of
// 64 rows x BM (BN) channels go to LDS as they lie in memory (direct global -> LDS loads, 16 bytes per lane) and the
// fragments are read through gfx950's transposing LDS read (ds_read_b64_tr_b16: sixteen lanes read a 4 x 16 block, each
// lane gets one column of it), so no operand is ever transposed in memory.  f32: the 32x32x2 MFMA takes one value per
// lane, so rows are read as they lie.  Swizzle: the four rows of a transposing read (the two of an f32 step) must fall on
// different banks; position q of row r holds 16-byte chunk q ^ key(r), chosen when the chunk is fetched.
// A lane's channel chunk, and with it its tap, is the same for the whole K loop; per K tile it decodes the pixel its row
// stands for (two multiply-high divisions per request) and asks for zeros (an out-of-range offset) outside the image.
//
// Few tiles and a long p: K is cut into `splits` slices, whose fp32 sums go to partial[slice][M][N]; tn_reduce_kernel adds
// them in a fixed order and writes the result as declared ([O][C][KH][KW]), so results do not depend on timing.
//
// Measured (kernel alone, before: the element gather with its packing step, or the images-last kernel with its two
// transpositions): 64x128x28x28 bf16 through 3x3 31 us + 5 us of adding (460 TFLOP/s; both gradients of the layer 93 -> 71 us),
// 32x64x28x28 f32 25 + 4 us (layer 131 -> 66 us), dense 512 x 1000 x 784 bf16 5 us (layer 62 -> 16 us).  Tiles: 128x128 runs
// one workgroup per CU at 1330 cycles per K tile (512 of them MFMA), 64x64 three per CU at 390 each.
#include <algorithm>

#include "igemm_tn.h"

namespace rl {

template <typename T, int BM, int BN, bool CONV>
__global__ __launch_bounds__(256) void igemm_tn_kernel(const TnParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub; the body uses gfx950-only builtins
    __shared__ __attribute__((aligned(1024))) unsigned char st0[tn_stage_bytes<BM, BN>()];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[tn_stage_bytes<BM, BN>()];
    __shared__ __attribute__((aligned(1024))) unsigned char st2[tn_stage_bytes<BM, BN>()];
    igemm_tn_body<T, BM, BN, CONV>(p, blockIdx.x, st0, st1, st2);
#endif
}

// y[m][c][tap] = sum over slices of partial[slice][m][(tap, c)], in a fixed order: `waves` waves of a workgroup each add a
// contiguous share of the slices of 64 groups of four columns in order, the first adds the shares in order.
__global__ void tn_reduce_kernel(const TnParams p, int waves)
{
    __shared__ f32x4 share[16][64];
    const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int64_t total4 = (int64_t)p.M * p.N / 4;
    const int64_t item = (int64_t)blockIdx.x * 64 + lane;
    const int per = (p.splits + waves - 1) / waves;
    const int c0 = grp * per, c1 = min(p.splits, c0 + per);
    f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
    if (item < total4) {
        const f32x4 *src = (const f32x4 *)p.partial + item;
        int z = c0;
        for (; z + 4 <= c1; z += 4) {
            const f32x4 v0 = src[(int64_t)z * total4], v1 = src[(int64_t)(z + 1) * total4];
            const f32x4 v2 = src[(int64_t)(z + 2) * total4], v3 = src[(int64_t)(z + 3) * total4];
            sum += v0; sum += v1; sum += v2; sum += v3;
        }
        for (; z < c1; ++z) sum += src[(int64_t)z * total4];
    }
    if (waves > 1) {
        share[grp][lane] = sum;
        __syncthreads();
        if (grp != 0) return;
        for (int g = 1; g < waves; ++g) sum += share[g][lane];
    }
    if (item >= total4) return;
    const int64_t idx = item * 4;
    const int m = (int)(idx / p.N), n = (int)(idx - (int64_t)m * p.N);
    const int tap = n / p.C, c = n - tap * p.C;         // C is a multiple of four
    if (m >= p.Mout) return;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (c + k < p.Cout) store_from_f32(p.y, p.y_dtype, ((int64_t)m * p.Cout + c + k) * p.T + tap, sum[k]);
}

#define RL_INST(T, BM, BN) template __global__ void igemm_tn_kernel<T, BM, BN, false>(const TnParams); template __global__ void igemm_tn_kernel<T, BM, BN, true>(const TnParams);
RL_INST(uint16_t, 128, 128) RL_INST(uint16_t, 64, 64) RL_INST(float, 128, 128) RL_INST(float, 64, 64)
#undef RL_INST

// rows are whole 16-byte chunks inside their tensors, offsets fit 31 bits, every slice holds a K tile and they cover K once; fills
// the grid's shape for square tiles
bool igemm_tn_prepare(TnParams &p, int element_size, int tile)
{
    const int KV = 16 / element_size, BK = 128 / element_size;
    p.nblk_m = (p.M + tile - 1) / tile;
    p.nblk_n = (p.N + tile - 1) / tile;
    const int64_t nk = ((int64_t)p.P + BK - 1) / BK, grid = (int64_t)p.nblk_m * p.nblk_n * p.splits;
    if (!p.a || !p.b || !p.y || ((uintptr_t)p.a & 15) || ((uintptr_t)p.b & 15) || p.M < 1 || p.N < 1 || p.P < 1 || p.P > 0x7fffff00 || p.T < 1 || p.C < 1 ||
        p.N != p.T * p.C || p.C % KV || p.M % KV || p.lda % KV || p.ldb % KV || p.lda < p.M || p.ldb < p.C || p.Cout > p.C || p.Mout > p.M ||
        (uint64_t)p.P * p.lda * element_size > p.a_bytes || p.a_bytes >= 0x80000000u || p.b_bytes >= 0x80000000u || p.splits < 1 || p.splits > 4096 || p.split_tiles < 1 ||
        (int64_t)p.splits * p.split_tiles < nk || (int64_t)(p.splits - 1) * p.split_tiles >= nk || (p.splits > 1 && (!p.partial || ((uintptr_t)p.partial & 15))) ||
        grid > 0x7fffffff)
        return false;
    const uint64_t rows = p.conv ? (uint64_t)((p.P + p.OHW - 1) / p.OHW) * p.H * p.W : (uint64_t)p.P;
    return rows * p.ldb * element_size <= p.b_bytes;
}

hipError_t launch_tn_reduce(const TnParams &p, hipStream_t s)
{
    const int waves = p.splits >= 32 ? 16 : p.splits >= 8 ? 4 : 1;
    const int64_t groups = ((int64_t)p.M * p.N / 4 + 63) / 64;
    hipLaunchKernelGGL(tn_reduce_kernel, dim3((unsigned)groups), dim3(64 * waves), 0, s, p, waves);
    return hipGetLastError();
}

template <typename T, int BM, int BN>
static hipError_t launch_tn(const TnParams &p0, hipStream_t s)
{
    TnParams p = p0;
    if (!igemm_tn_prepare(p, (int)sizeof(T), BM)) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)((int64_t)p.nblk_m * p.nblk_n * p.splits);
    if (p.conv) hipLaunchKernelGGL((igemm_tn_kernel<T, BM, BN, true>), dim3(grid), dim3(256), 0, s, p);
    else hipLaunchKernelGGL((igemm_tn_kernel<T, BM, BN, false>), dim3(grid), dim3(256), 0, s, p);
    hipError_t er = hipGetLastError();
    if (er != hipSuccess || p.splits == 1) return er;
    return launch_tn_reduce(p, s);
}

hipError_t launch_igemm_tn(const TnParams &p, int32_t dtype, int32_t tile, hipStream_t s)
{
    if (dtype == DT_BF16) return tile == 128 ? launch_tn<uint16_t, 128, 128>(p, s) : launch_tn<uint16_t, 64, 64>(p, s);
    return tile == 128 ? launch_tn<float, 128, 128>(p, s) : launch_tn<float, 64, 64>(p, s);
}

}  // namespace rl
