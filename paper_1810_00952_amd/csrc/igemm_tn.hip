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

#include "device_utils.h"

namespace rl {

namespace {

typedef __amdgpu_buffer_rsrc_t rsrc_t;
#define RL_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

__device__ __forceinline__ rsrc_t make_rsrc(const void *ptr, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)ptr, 0, bytes, 0x00020000);   // raw buffer, untyped dwords
}

// The wave's direct loads but the last N have landed and its own LDS reads are done (so that nobody's next direct load can
// overtake them), then the workgroup barrier; nothing moves across.
template <int N> __device__ __forceinline__ void wait_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

// n / d for n < 2^31; d == 1 comes as mul = 0, sh = 0 and an all-ones mask (no branch in the K loop)
__device__ __forceinline__ uint32_t fast_div(uint32_t n, uint32_t mul, uint32_t sh, uint32_t one)
{
    return (__umulhi(n, mul) + (n & one)) >> sh;
}

constexpr int NUM_XCD = 8;
constexpr uint32_t OOB = 0x80000000u;

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

// key(r) of the swizzle, in chunks.  bf16: a transposing read touches rows r .. r+3 (r a multiple of 4) at the same 64 bytes;
// f32: a step reads rows r, r+1 (r even) at the same 128 bytes.  A row of 128 bytes shares its 256-byte line with a neighbour.
template <int ES, int ROWB> __device__ __forceinline__ int swz(int r)
{
    if (ES == 2) return ROWB == 256 ? (r & 3) << 2 : ((r >> 1) & 1) << 2;
    return (r & 1) << 3;
}

}  // namespace

template <typename T, int BM, int BN, bool CONV>
__global__ __launch_bounds__(256) void igemm_tn_kernel(const TnParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub; the body uses gfx950-only builtins
    constexpr int ES = (int)sizeof(T), KV = 16 / ES;
    constexpr int BK = ES == 2 ? 64 : 32;             // rows (pixels) per K tile
    constexpr int WTM = BM / 2, WTN = BN / 2, TM = WTM / 32, TN = WTN / 32;
    constexpr int ROWA = BM * ES, ROWB = BN * ES;     // bytes per LDS row
    constexpr int A_BYTES = BK * ROWA, B_BYTES = BK * ROWB, STAGE = A_BYTES + B_BYTES;
    constexpr int AG = A_BYTES / 4096, BG = B_BYTES / 4096;   // direct loads per wave and tile
    constexpr int RA = 1024 / ROWA, RB = 1024 / ROWB; // rows per direct load
    constexpr int LPT = AG + BG;

    __shared__ __attribute__((aligned(1024))) unsigned char st0[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st2[STAGE];

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // workgroups of one slice share its rows of A and B: slices in order, each XCD a contiguous run
    const int tiles = p.nblk_m * p.nblk_n, nblk = tiles * p.splits;
    int bid = blockIdx.x;
    {
        const int per = nblk / NUM_XCD, main = per * NUM_XCD;
        if (bid < main) bid = (bid % NUM_XCD) * per + bid / NUM_XCD;
    }
    const int split = bid / tiles, tile = bid - split * tiles;
    const int bm = tile / p.nblk_n, bn = tile - bm * p.nblk_n;
    const int m0 = bm * BM, n0 = bn * BN;
    const int nk_all = (p.P + BK - 1) / BK;
    const int kt0 = split * p.split_tiles, nk = min(nk_all, kt0 + p.split_tiles);

    const rsrc_t ra = make_rsrc(p.a, p.a_bytes), rb = make_rsrc(p.b, p.b_bytes);

    // ---- what this lane requests: rows (kt BK + a_row + RA i) of A at one chunk of channels, likewise of B at one (tap, chunk)
    const int a_row = wave * AG * RA + lane / (ROWA / 16);
    const int b_row = wave * BG * RB + lane / (ROWB / 16);
    const int a_col = m0 + ((lane % (ROWA / 16)) ^ swz<ES, ROWA>(a_row)) * KV;
    const int b_col = n0 + ((lane % (ROWB / 16)) ^ swz<ES, ROWB>(b_row)) * KV;
    const bool a_in = a_col < p.M, b_in = b_col < p.N;
    const uint32_t lda = (uint32_t)p.lda * ES, ldb = (uint32_t)p.ldb * ES;
    const uint32_t a_off = (uint32_t)a_col * ES;
    int dh = 0, dw = 0;
    uint32_t b_off = (uint32_t)b_col * ES;
    if (CONV) {
        const int tap = b_col / p.C, kh = tap / p.KW;
        b_off = (uint32_t)(b_col - tap * p.C) * ES;
        dh = kh - p.ph;
        dw = tap - kh * p.KW - p.pw;
    }

    const uint32_t one_ohw = p.OHW == 1 ? ~0u : 0u, one_ow = p.OW == 1 ? ~0u : 0u;
    int f_row = kt0 * BK;                              // first row of the tile requested next
    const int row_end = min(p.P, nk * BK);
#define RL_ISSUE(ST)                                                                                                  \
    {                                                                                                                 \
        _Pragma("unroll") for (int i = 0; i < AG; ++i) {                                                              \
            const int r = f_row + a_row + RA * i;                                                                     \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, RL_LDS_PTR(ST + (wave * AG + i) * 1024), 16,                 \
                                                     a_in && r < row_end ? (uint32_t)r * lda + a_off : OOB, 0, 0, 0); \
        }                                                                                                             \
        _Pragma("unroll") for (int i = 0; i < BG; ++i) {                                                              \
            const int r = f_row + b_row + RB * i;                                                                     \
            bool ok = b_in && r < row_end;                                                                            \
            uint32_t row = (uint32_t)r;                                                                               \
            if (CONV) {                                                                                               \
                const int img = (int)fast_div((uint32_t)r, p.div_ohw_mul, p.div_ohw_sh, one_ohw);                      \
                const int pix = r - img * p.OHW;                                                                      \
                const int oh = (int)fast_div((uint32_t)pix, p.div_ow_mul, p.div_ow_sh, one_ow);                        \
                const int ih = oh * p.s + dh, iw = (pix - oh * p.OW) * p.s + dw;                                      \
                ok = ok && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;                              \
                row = (uint32_t)((img * p.H + ih) * p.W + iw);                                                        \
            }                                                                                                         \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, RL_LDS_PTR(ST + A_BYTES + (wave * BG + i) * 1024), 16,       \
                                                     ok ? row * ldb + b_off : OOB, 0, 0, 0);                          \
        }                                                                                                             \
        f_row += BK;                                                                                                  \
    }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // ---- fragment addresses inside a tile
    int fa[TM], fb[TN];
    if (ES == 2) {
        const int g = lane >> 4, q = lane & 15;        // lane q of a group of sixteen reads row q / 4 of the group's block, columns 4 (q & 3) ..
        const int kr = (g >> 1) * 8 + (q >> 2), cc = (g & 1) * 2 + ((q & 3) >> 1), half = (q & 1) * 8;
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i] = kr * ROWA + ((((wm * WTM + i * 32) / 8 + cc) ^ swz<ES, ROWA>(kr)) << 4) + half;
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[j] = kr * ROWB + ((((wn * WTN + j * 32) / 8 + cc) ^ swz<ES, ROWB>(kr)) << 4) + half;
    } else {
        const int kr = lane >> 5, cl = lane & 31;
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i] = kr * ROWA + ((((wm * WTM + i * 32 + cl) / 4) ^ swz<ES, ROWA>(kr)) << 4) + (cl & 3) * 4;
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[j] = kr * ROWB + ((((wn * WTN + j * 32 + cl) / 4) ^ swz<ES, ROWB>(kr)) << 4) + (cl & 3) * 4;
    }

    auto tr8 = [](const unsigned char *base, int off, int row4) -> bf16x8 {      // eight contraction indices of the lane's column
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(base + off));
        s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(base + off + row4));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto compute = [&](const unsigned char *st) {
        if constexpr (ES == 2) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                bf16x8 va[TM], vb[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i) va[i] = tr8(st, fa[i] + ks * 16 * ROWA, 4 * ROWA);
#pragma unroll
                for (int j = 0; j < TN; ++j) vb[j] = tr8(st, A_BYTES + fb[j] + ks * 16 * ROWB, 4 * ROWB);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i], vb[j], acc[i][j], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int ks = 0; ks < 16; ++ks) {
                float va[TM], vb[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i) va[i] = *(const float *)(st + fa[i] + ks * 2 * ROWA);
#pragma unroll
                for (int j = 0; j < TN; ++j) vb[j] = *(const float *)(st + A_BYTES + fb[j] + ks * 2 * ROWB);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[i], vb[j], acc[i][j], 0, 0, 0);
            }
        }
    };

    // ---- K loop, three stages: wait for this wave's part of tile kt (the requests of tile kt+1 may still fly), barrier,
    // request tile kt+2 into the stage tile kt-1 just left, multiply tile kt.  Requests past the slice are out of range.
#define RL_BODY(CUR, NXT)     \
    {                         \
        wait_barrier<LPT>();  \
        RL_ISSUE(NXT)         \
        compute(CUR);         \
    }
    RL_ISSUE(st0)
    RL_ISSUE(st1)
    int kt = kt0;
#pragma unroll 1
    for (; kt + 3 <= nk; kt += 3) {
        RL_BODY(st0, st2)
        RL_BODY(st1, st0)
        RL_BODY(st2, st1)
    }
    if (kt < nk) {
        RL_BODY(st0, st2)
        if (kt + 1 < nk) RL_BODY(st1, st0)
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // the trailing out-of-range requests
#undef RL_BODY
#undef RL_ISSUE

    // ---- register 4g + k of lane l holds row 8g + 4 (l >> 5) + k, column l & 31 of its 32 x 32 tile
    const int col = lane & 31, fhalf = lane >> 5;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = n0 + wn * WTN + j * 32 + col;
        if (n >= p.N) continue;
        const int tap = CONV ? n / p.C : 0, c = n - tap * p.C;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + wm * WTM + i * 32 + 8 * (r >> 2) + 4 * fhalf + (r & 3);
                if (m >= p.M) continue;
                if (p.splits > 1) p.partial[((int64_t)split * p.M + m) * p.N + n] = acc[i][j][r];
                else if (c < p.Cout && m < p.Mout) store_from_f32(p.y, p.y_dtype, ((int64_t)m * p.Cout + c) * p.T + tap, acc[i][j][r]);
            }
    }
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

template <typename T, int BM, int BN>
static hipError_t launch_tn(const TnParams &p0, hipStream_t s)
{
    TnParams p = p0;
    constexpr int KV = 16 / (int)sizeof(T), BK = 128 / (int)sizeof(T);
    p.nblk_m = (p.M + BM - 1) / BM;
    p.nblk_n = (p.N + BN - 1) / BN;
    const int64_t nk = ((int64_t)p.P + BK - 1) / BK, grid = (int64_t)p.nblk_m * p.nblk_n * p.splits;
    // rows are whole 16-byte chunks inside their tensors, offsets fit 31 bits, every slice holds a K tile and they cover K once
    if (!p.a || !p.b || !p.y || ((uintptr_t)p.a & 15) || ((uintptr_t)p.b & 15) || p.M < 1 || p.N < 1 || p.P < 1 || p.P > 0x7fffff00 || p.T < 1 || p.C < 1 ||
        p.N != p.T * p.C || p.C % KV || p.M % KV || p.lda % KV || p.ldb % KV || p.lda < p.M || p.ldb < p.C || p.Cout > p.C || p.Mout > p.M ||
        (uint64_t)p.P * p.lda * sizeof(T) > p.a_bytes || p.a_bytes >= 0x80000000u || p.b_bytes >= 0x80000000u || p.splits < 1 || p.splits > 4096 || p.split_tiles < 1 ||
        (int64_t)p.splits * p.split_tiles < nk || (int64_t)(p.splits - 1) * p.split_tiles >= nk || (p.splits > 1 && (!p.partial || ((uintptr_t)p.partial & 15))) ||
        grid > 0x7fffffff)
        return hipErrorInvalidValue;
    const uint64_t rows = p.conv ? (uint64_t)((p.P + p.OHW - 1) / p.OHW) * p.H * p.W : (uint64_t)p.P;
    if (rows * p.ldb * sizeof(T) > p.b_bytes) return hipErrorInvalidValue;
    if (p.conv) hipLaunchKernelGGL((igemm_tn_kernel<T, BM, BN, true>), dim3((unsigned)grid), dim3(256), 0, s, p);
    else hipLaunchKernelGGL((igemm_tn_kernel<T, BM, BN, false>), dim3((unsigned)grid), dim3(256), 0, s, p);
    hipError_t er = hipGetLastError();
    if (er != hipSuccess || p.splits == 1) return er;
    const int waves = p.splits >= 32 ? 16 : p.splits >= 8 ? 4 : 1;
    const int64_t groups = ((int64_t)p.M * p.N / 4 + 63) / 64;
    hipLaunchKernelGGL(tn_reduce_kernel, dim3((unsigned)groups), dim3(64 * waves), 0, s, p, waves);
    return hipGetLastError();
}

hipError_t launch_igemm_tn(const TnParams &p, int32_t dtype, int32_t tile, hipStream_t s)
{
    if (dtype == DT_BF16) return tile == 128 ? launch_tn<uint16_t, 128, 128>(p, s) : launch_tn<uint16_t, 64, 64>(p, s);
    return tile == 128 ? launch_tn<float, 128, 128>(p, s) : launch_tn<float, 64, 64>(p, s);
}

}  // namespace rl
