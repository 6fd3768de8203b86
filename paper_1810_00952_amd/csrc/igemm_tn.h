// The workgroup of the contraction over the rows of both operands (igemm_tn.hip, where its design is described), for the kernels
// that run it alone or beside another contraction (igemm_grads.hip).
#pragma once
#include "igemm_lds.h"

namespace rl {

namespace {

// n / d for n < 2^31; d == 1 comes as mul = 0, sh = 0 and an all-ones mask (no branch in the K loop)
__device__ __forceinline__ uint32_t fast_div(uint32_t n, uint32_t mul, uint32_t sh, uint32_t one)
{
    return (__umulhi(n, mul) + (n & one)) >> sh;
}

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

// Tile and K slice `bid` (numbered for the XCDs) by the 256 threads of a workgroup; st0 .. st2: its LDS
template <int BM, int BN> constexpr int tn_stage_bytes() { return (BM + BN) * 128; }       // 64 bf16 or 32 f32 rows
template <typename T, int BM, int BN, bool CONV>
__device__ __forceinline__ void igemm_tn_body(const TnParams &p, int bid, unsigned char (&st0)[tn_stage_bytes<BM, BN>()], unsigned char (&st1)[tn_stage_bytes<BM, BN>()],
                                              unsigned char (&st2)[tn_stage_bytes<BM, BN>()])
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

    static_assert(STAGE == tn_stage_bytes<BM, BN>(), "a stage");

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // workgroups of one slice share its rows of A and B: slices in order, each XCD a contiguous run
    const int tiles = p.nblk_m * p.nblk_n;
    bid = xcd_run(bid, tiles * p.splits);
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
    // f32 on 64x64 tiles: the sums of twelve K tiles (384 rows) are added to those of the rows before them, so that a long slice is not one
    // serial sum (32x64x28x28, slices of 20 K tiles: 4.5e-7 from the value in 64 bits without, 4.2e-7 with; slices of 10 without 4.2e-7)
    constexpr bool LEVELS = ES == 4 && TM == 1 && TN == 1;
    f32x16 sums;
    if constexpr (LEVELS) {
#pragma unroll
        for (int e = 0; e < 16; ++e) sums[e] = 0.0f;
    }
    auto carry = [&]() {
        if constexpr (LEVELS) {
#pragma unroll
            for (int e = 0; e < 16; ++e) { sums[e] += acc[0][0][e]; acc[0][0][e] = 0.0f; }
        }
    };
    RL_ISSUE(st0)
    RL_ISSUE(st1)
    int kt = kt0, level = 0;
#pragma unroll 1
    for (; kt + 3 <= nk; kt += 3) {
        RL_BODY(st0, st2)
        RL_BODY(st1, st0)
        RL_BODY(st2, st1)
        if (LEVELS && ++level == 4) {
            carry();
            level = 0;
        }
    }
    if (kt < nk) {
        RL_BODY(st0, st2)
        if (kt + 1 < nk) RL_BODY(st1, st0)
    }
    carry();
    if constexpr (LEVELS) acc[0][0] = sums;
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

}  // namespace rl
