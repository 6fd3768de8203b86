// The direct-load contraction kernel (igemm_dma.hip, where its design is described), alone in its grid or beside another contraction
// (igemm_grads.hip).
#pragma once
#include "igemm_epilogue.h"
#include "igemm_lds.h"

namespace rl {

namespace {

__device__ __forceinline__ void mma_chunk(f32x16 &acc, const u32x4 &a, const u32x4 &b, float)
{
#pragma unroll
    for (int j = 0; j < 4; ++j)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[j]), __uint_as_float(b[j]), acc, 0, 0, 0);
}

__device__ __forceinline__ void mma_chunk(f32x16 &acc, const u32x4 &a, const u32x4 &b, uint16_t)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

__device__ __forceinline__ void wg_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

}  // namespace

// MODE of the result: rows of channels 16 bytes at a time, the LSTM gates, or any order
enum { STORE_ROWS = 0, STORE_GATES = 1, STORE_ANY = 2 };

// TEAMS: 2: eight waves, of which each half takes two of the four steps of every K tile; the halves' sums meet at the end.  With one workgroup
// on a CU a K tile is a serial chain per wave (four direct loads, eight fragment reads, the MFMAs, the barrier: 690 cycles, however
// many tiles are requested ahead).  Each wave then has half of the loads, reads and MFMAs; the latency of each link and the barrier stay, and
// of the 690 cycles about 45 go (13 K tiles, the meeting of the sums included).  Grids of at most 256 workgroups without K slices (82 drawn dense layers 0.95 to 0.99 of
// their time by the number of K tiles; slices, whose K tiles are two or three, would lose 2 %): dense 1000 x 1000 x 784 bf16 8.04 -> 7.76 us,
// 4x96x29x29 -> 136 3x3 with a residual 17.9 -> 16.3; 17 images (672 workgroups, which cover each other's chains) 24.4 against 26.8.
// BESIDE: the workgroups of another contraction in the same grid (igemm_grads.hip).  Its take() does the work of those and returns false,
// or returns true with the number of this contraction's workgroup.
struct Alone {
    static constexpr bool other = false;
};

// The body is the kernel's own text and no function that takes its arguments by reference: inlined from one, the compiler no longer holds
// them for constant memory while it orders the code, and fetches those of the epilogue one by one, each where it is used (17 more scalar
// loads; dense 1000 x 1000 x 784 bf16 8.2 us against 7.95, 17x96x29x29 -> 136 3x3 with a residual 21.8 against 21.4).
template <int BM, int BN> constexpr int dma_stage_bytes() { return (BM + BN) * 128; }
template <typename T, int BM, int BN, int MODE, bool TAPS, typename BESIDE, int TEAMS>
__global__ __launch_bounds__(256 * TEAMS) void igemm_dma_kernel(const IgemmParams p, const BESIDE beside)
{
    constexpr bool GATES = MODE == STORE_GATES;
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub; the body uses gfx950-only builtins
    __shared__ __attribute__((aligned(1024))) unsigned char st0[dma_stage_bytes<BM, BN>()];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[dma_stage_bytes<BM, BN>()];
    __shared__ __attribute__((aligned(1024))) unsigned char st2[dma_stage_bytes<BM, BN>()];
    int bid = blockIdx.x, split = 0;
    if constexpr (BESIDE::other) {
        if (!beside.template take<T>(bid, st0, st1, st2)) return;
        const int tiles = p.nblk_m * p.nblk_n;
        if (bid >= tiles * max(p.splits, 1)) return;
        split = p.splits > 1 ? bid / tiles : 0;
        bid -= split * tiles;
    } else {
        split = p.splits > 1 ? (int)blockIdx.y : 0;
    }
    touch_args(p);
    constexpr int KV = Elem<T>::KV;
    constexpr int ES = (int)sizeof(T);
    constexpr int BKE = 8 * KV;               // K elements per tile (128 bytes per row)
    constexpr int WTM = BM / 2, WTN = BN / 2; // wave tile
    constexpr int TM = WTM / 32, TN = WTN / 32;
    constexpr int AG = BM / 32 / TEAMS, BG = BN / 32 / TEAMS; // 8-row DMA groups per wave
    constexpr int KS = 4 / TEAMS;             // of the four steps of a K tile, a team's own
    constexpr int LPT = AG + BG;              // DMA instructions per wave per tile
    constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128, STAGE = A_BYTES + B_BYTES;
    constexpr int LDC = BN + 8;               // fp32 staging row (32 rows at a time)
    static_assert(32 * LDC * 4 <= STAGE, "epilogue staging must fit in one stage");

    const int t = threadIdx.x & 255;          // within the team
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);   // wave-uniform by construction; keep it in an SGPR
    const int team = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;

    // The kernel arguments that the first request hangs on, fetched together; left to itself the compiler asks for some of them
    // behind the arithmetic on others (dense 1000 x 1000 x 784 bf16 8.94 -> 8.62 us, two-layer classifier f32 12.52 -> 12.43); the lines
    // of all others above (8.24 -> 7.97; dense gradients, each a launch, 15.48 -> 15.07).  The longer kernels do not gain by it.
    asm volatile("" :: "s"(p.nblk_m), "s"(p.nblk_n), "s"(p.x), "s"(p.w), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.Kp), "s"(p.K1), "s"(p.C), "s"(p.H), "s"(p.W), "s"(p.KH), "s"(p.KW),
                 "s"(p.OW), "s"(p.OHW), "s"(p.sh), "s"(p.sw), "s"(p.ph), "s"(p.pw), "s"(p.xs_n), "s"(p.xs_h), "s"(p.xs_w), "s"(p.x_bytes), "s"(p.w_bytes), "s"(p.splits), "s"(p.split_tiles), "s"(p.div_ohw_mul), "s"(p.div_ohw_sh), "s"(p.div_ow_mul), "s"(p.div_ow_sh));
    bid = xcd_run(bid, p.nblk_m * p.nblk_n);
    const int bm = bid / p.nblk_n, bn = bid - bm * p.nblk_n;
    const int m0 = bm * BM, n0 = bn * BN;

    // The activation descriptor starts `bias` bytes before x so that the per-lane offset of a
    // row's tap (0,0) -- which lies above/left of the image for border pixels -- is never negative.
    const uint32_t bias = (uint32_t)(((int64_t)p.ph * p.xs_h + (int64_t)p.pw * p.xs_w) * ES);
    const rsrc_t rx = make_rsrc((const char *)p.x - bias, p.x_bytes + bias);
    const rsrc_t rx2 = make_rsrc(p.x2 ? p.x2 : p.x, p.x2 ? p.x2_bytes : p.x_bytes);
    const rsrc_t rw = make_rsrc(p.w, p.w_bytes);

    // ---- per-lane DMA state.  Lane l of a group writes LDS row (l >> 3), position (l & 7).
    const int r8 = lane >> 3, pos = lane & 7;
    uint32_t a_voff[AG], a_mask[AG], a2_voff[AG], b_voff[BG];
    int a_kc[AG];                       // first K element (within a tile) of the 16-byte chunk this lane fetches
    int t_ih[AG], t_iw[AG];             // TAPS: input coordinate of tap (0, 0)
    static_assert((AG % 2 == 0 && BG % 2 == 0) || (AG == 1 && BG == 1), "a lane's chunk depends on the parity of its row group only");
    constexpr int PAR = AG == 1 ? 1 : 2;
#pragma unroll
    for (int i = 0; i < AG; ++i) {
        const int row = wave * 8 * AG + 8 * i + r8;
        const int chunk = pos ^ ((row >> 1) & 7);
        const int m = m0 + row;
        uint32_t mask = 0;
        int64_t off = 0;
        if (m < p.M) {
            // by multiply-high: dense 1000 x 1000 x 784 bf16 8.36 -> 8.04 us, LeNet's shape 28.0 -> 27.6
            const int img = p.OHW == 1 ? m : (int)(__umulhi((uint32_t)m, p.div_ohw_mul) >> p.div_ohw_sh);
            const int pix = m - img * p.OHW;
            const int oh = p.OW == 1 ? pix : (int)(__umulhi((uint32_t)pix, p.div_ow_mul) >> p.div_ow_sh);
            const int ow = pix - oh * p.OW;
            int ih0 = oh * p.sh - p.ph, iw0 = ow * p.sw - p.pw;
            t_ih[i] = ih0; t_iw[i] = iw0;
            if (!TAPS)
            for (int kh = 0; kh < p.KH; ++kh)
                for (int kw = 0; kw < p.KW; ++kw)
                    mask |= (uint32_t)(((unsigned)(ih0 + kh) < (unsigned)p.H) & ((unsigned)(iw0 + kw) < (unsigned)p.W)) << (kh * p.KW + kw);      // without a branch: ResNet-18 shape, one image f32, 257.5 -> 253.4 us
            off = ((int64_t)img * p.xs_n + (int64_t)ih0 * p.xs_h + (int64_t)iw0 * p.xs_w) * ES;
        }
        if (m >= p.M) { t_ih[i] = -(1 << 24); t_iw[i] = 0; }
        a_mask[i] = mask;
        a_kc[i] = chunk * KV;
        a_voff[i] = (uint32_t)(off + bias) + (TAPS ? 0 : chunk * 16);
        a2_voff[i] = (uint32_t)((int64_t)m * p.x2s_n * ES) + chunk * 16;     // second operand of a concatenation: row m
    }
#pragma unroll
    for (int j = 0; j < BG; ++j) {
        const int row = wave * 8 * BG + 8 * j + r8;
        const int chunk = pos ^ ((row >> 1) & 7);
        int n = n0 + row;
        if (n > p.N - 1) n = p.N - 1;          // rows past N are computed on valid memory and never stored
        b_voff[j] = (uint32_t)((int64_t)n * p.Kp * ES) + (TAPS ? 0 : chunk * 16);
    }
    const uint32_t one_c = p.C == 1 ? ~0u : 0u, one_kw = p.KW == 1 ? ~0u : 0u;

    // ---- wave-uniform K state of the tile to be issued next.  Issuing is unconditional so that
    // every K-loop body has the same number of DMA instructions in flight (the explicit vmcnt
    // waits count on it); past the last tile all lanes are sent out of range, which costs no
    // memory traffic and only zero-fills a stage nobody reads.
    // K tiles [kt0, nk) of the contraction's ceil(p.K / BKE) (>= 2): all of them, or this workgroup's slice.  Only a
    // one-tap contraction (dense, 1x1) may end in a partial tile: the weights are packed with zeros up to the tile,
    // the activation chunks past K are requested out of range.
    const int nk_all = (p.K + BKE - 1) / BKE;
    const int kt0 = p.splits > 1 ? split * p.split_tiles : 0;
    const int nk = p.splits > 1 ? min(nk_all, kt0 + p.split_tiles) : nk_all;
    int f_kt = kt0, f_c0 = 0, f_tap = 0, f_kh = 0, f_kw = 0;
    if (!TAPS && kt0 > 0) {
        const int tpt = p.KH * p.KW == 1 ? nk_all : p.C / BKE;      // K tiles per filter tap
        f_tap = kt0 / tpt;
        f_c0 = (kt0 - f_tap * tpt) * BKE;
        f_kh = f_tap / p.KW;
        f_kw = f_tap - f_kh * p.KW;
    }
#define RL_ISSUE_UNIFORM(ST)                                                                                                  \
    {                                                                                                                 \
        const bool live = f_kt < nk;                                                                                  \
        const int k0 = f_kt * BKE;                                                                                    \
        const uint32_t soff_b = live ? (uint32_t)k0 * ES : 0u;                                                        \
        if (k0 < p.K1 || !live) {                                                                                     \
            const uint32_t tapbit = live ? (1u << f_tap) : 0u;                                                        \
            const uint32_t soff_a = live ? (uint32_t)(((int64_t)f_kh * p.xs_h + (int64_t)f_kw * p.xs_w + f_c0) * ES) : 0u; \
            const int krem = p.K - k0;      /* K elements from this tile's start on: >= BKE except in a partial last tile */ \
            _Pragma("unroll") for (int i = 0; i < AG; ++i)                                                            \
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, RL_LDS_PTR(ST + (wave * AG + i) * 1024), 16,             \
                                                         ((a_mask[i] & tapbit) && a_kc[i] < krem) ? a_voff[i] : OOB, soff_a, 0, 0); \
        } else {                                                                                                      \
            const uint32_t soff_a = (uint32_t)(k0 - p.K1) * ES;                                                       \
            _Pragma("unroll") for (int i = 0; i < AG; ++i)                                                            \
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rx2, RL_LDS_PTR(ST + (wave * AG + i) * 1024), 16,            \
                                                         a_mask[i] ? a2_voff[i] : OOB, soff_a, 0, 0);                 \
        }                                                                                                             \
        _Pragma("unroll") for (int j = 0; j < BG; ++j)                                                                \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, RL_LDS_PTR(ST + A_BYTES + (wave * BG + j) * 1024), 16,       \
                                                     live ? b_voff[j] : OOB, soff_b, 0, 0);                           \
        ++f_kt;                                                                                                       \
        f_c0 += BKE;                                                                                                  \
        if (f_c0 >= p.C) {                                                                                            \
            f_c0 = 0;                                                                                                 \
            ++f_tap;                                                                                                  \
            if (++f_kw == p.KW) { f_kw = 0; ++f_kh; }                                                                 \
        }                                                                                                             \
    }

#define RL_ISSUE_TAPS(ST)                                                                                             \
    {                                                                                                                 \
        const bool live = f_kt < nk;                                                                                  \
        uint32_t toff[PAR], koff[PAR];                                                                                \
        int tkh[PAR], tkw[PAR];                                                                                       \
        bool oka[PAR], okb[PAR];                                                                                      \
        _Pragma("unroll") for (int e = 0; e < PAR; ++e) {                                                             \
            const uint32_t k = (uint32_t)(f_kt * BKE + a_kc[e]);                                                      \
            const uint32_t tap = (__umulhi(k, p.div_c_mul) + (k & one_c)) >> p.div_c_sh;                              \
            tkh[e] = (int)((__umulhi(tap, p.div_kw_mul) + (tap & one_kw)) >> p.div_kw_sh);                            \
            tkw[e] = (int)tap - tkh[e] * p.KW;                                                                        \
            toff[e] = (uint32_t)(((int)k - (int)tap * p.C + tkh[e] * (int)p.xs_h + tkw[e] * (int)p.xs_w) * ES);       \
            koff[e] = k * ES;                                                                                         \
            oka[e] = live && k < (uint32_t)p.K;                                                                       \
            okb[e] = live && k < (uint32_t)p.Kp;                                                                      \
        }                                                                                                             \
        _Pragma("unroll") for (int i = 0; i < AG; ++i) {                                                              \
            const int e = i & 1;                                                                                      \
            const bool ok = oka[e] && (unsigned)(t_ih[i] + tkh[e]) < (unsigned)p.H && (unsigned)(t_iw[i] + tkw[e]) < (unsigned)p.W; \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, RL_LDS_PTR(ST + (wave * AG + i) * 1024), 16, ok ? a_voff[i] + toff[e] : OOB, 0, 0, 0); \
        }                                                                                                             \
        _Pragma("unroll") for (int j = 0; j < BG; ++j)                                                                \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, RL_LDS_PTR(ST + A_BYTES + (wave * BG + j) * 1024), 16,       \
                                                     okb[j & 1] ? b_voff[j] + koff[j & 1] : OOB, 0, 0, 0);            \
        ++f_kt;                                                                                                       \
    }

#define RL_ISSUE(ST) { if constexpr (TAPS) RL_ISSUE_TAPS(ST) else RL_ISSUE_UNIFORM(ST) }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // ---- fragment addresses: row frow of a 32-row MFMA tile, chunk 2*ks + fhalf, swizzled
    const int frow = lane & 31, fhalf = lane >> 5;
    int f_off[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) f_off[ks] = frow * 128 + (((2 * (team * KS + ks) + fhalf) ^ ((frow >> 1) & 7)) << 4);

    // All of a tile's reads before its first MFMA: they are done while the MFMAs run, and the wait before the next barrier costs nothing.
#define RL_COMPUTE(ST)                                                                                                \
    {                                                                                                                 \
        u32x4 fa[KS][TM], fb[KS][TN];                                                                                 \
        _Pragma("unroll") for (int ks = 0; ks < KS; ++ks) {                                                           \
            _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                            \
                fa[ks][i] = *(const u32x4 *)(ST + (wm * WTM + i * 32) * 128 + f_off[ks]);                             \
            _Pragma("unroll") for (int j = 0; j < TN; ++j)                                                            \
                fb[ks][j] = *(const u32x4 *)(ST + A_BYTES + (wn * WTN + j * 32) * 128 + f_off[ks]);                   \
        }                                                                                                             \
        __builtin_amdgcn_sched_barrier(0);                                                                            \
        _Pragma("unroll") for (int ks = 0; ks < KS; ++ks)                                                             \
            _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                            \
                _Pragma("unroll") for (int j = 0; j < TN; ++j) mma_chunk(acc[i][j], fa[ks][i], fb[ks][j], T());       \
    }

    // Results in Shape order: the epilogue's operands of a thread's pixels, requested ahead of the K loop (they arrive under it; asked for
    // where they are needed, pass by pass, they were most of a short contraction's time).
    // 17x96x29x29 -> 136 3x3 bf16 with a residual 25.5 -> 21.6 us; 130 bf16 layers 0.93 (128x64) and 0.98, f32 on 128x64 0.97, on 64x64
    // level and left as it was.  (128x128: too many registers.)
    constexpr bool AHEAD = MODE == STORE_ANY && BM * BN <= 128 * 64 && (ES == 2 || BM == 128);
    PixelEpilogue<AHEAD ? BM : 32, AHEAD ? BN : 32> pe;
    pe.form = PE_NONE;
    if constexpr (AHEAD) if (team == 0) pe.request(p, t, m0, n0);
    using TE = TileEpilogue<BN>;
    const bool pre = !GATES && p.epi.simple;
    float bias8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    OperandRegs<TE::NV> cur = {}, nxt = {};
    auto request_rows = [&]() {
        if (!pre) return;
        TE::load_bias(p, t, n0, bias8);
        TE::prefetch(p, t, m0, n0, cur);
    };
    if constexpr (TEAMS > 1 && MODE == STORE_ROWS) if (team == 0) request_rows();

    // ---- K loop, three stages, unrolled by three so that every stage use names its array.
    // Tile kt lives in stage kt % 3.  Body: wait until my DMAs of tile kt have landed (the LPT
    // issued after them, for tile kt+1, may still fly) and my reads of tile kt-1 are done, barrier, issue tile kt+2 into the stage
    // tile kt-1 just left, MFMAs on tile kt.
#define RL_BODY(CUR, NXT)     \
    {                         \
        wait_barrier<LPT>();  \
        RL_ISSUE(NXT)         \
        RL_COMPUTE(CUR)       \
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
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");           // the trailing out-of-range issues, the last tile's reads
#undef RL_BODY
#undef RL_COMPUTE
#undef RL_ISSUE
#undef RL_ISSUE_TAPS
#undef RL_ISSUE_UNIFORM

    if constexpr (TEAMS > 1) {
        // the second team's sums into stage 1's array, and to the first team's
        static_assert(TEAMS == 2 && TM == 1 && TN == 1 && STAGE == 4 * 64 * 64, "a stage holds a team's sums");
        f32x4 *sums = (f32x4 *)st1 + (wave & 3) * 4 * 64 + lane;
        wg_barrier();                               // every wave's direct loads and reads are done
        if (team == 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) sums[r * 64] = f32x4{acc[0][0][4 * r], acc[0][0][4 * r + 1], acc[0][0][4 * r + 2], acc[0][0][4 * r + 3]};
        }
        __syncthreads();
        if (team == 1) return;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const f32x4 v = sums[r * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[0][0][4 * r + e] += v[e];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // read out before the barrier behind which stage 1 is written again
    }

    // ---- epilogue: 32 rows at a time through LDS (stage 0's array), then 8 channels per thread;
    // the residual rows of the next pass are fetched while this pass is staged and stored
    float *sC = (float *)st0;
    if (MODE == STORE_ROWS && p.splits > 1) {
        // a slice of K: the bare fp32 sums, row-major [M][N], into this slice's part of the scratch tensor
        float *dst = p.partial + (int64_t)split * p.M * p.N;
#pragma unroll
        for (int q = 0; q < BM / 32; ++q) {
            wg_barrier();
            if (wm == q / TM) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        int row = 8 * (r >> 2) + 4 * fhalf + (r & 3);
                        int col = wn * WTN + j * 32 + frow;
                        sC[row * LDC + col] = acc[q % TM][j][r];
                    }
            }
            __syncthreads();
            for (int idx = t; idx < 32 * BN; idx += 256) {
                const int row = idx / BN, col = idx - row * BN;
                const int m = m0 + q * 32 + row, n = n0 + col;
                if (m < p.M && n < p.N) dst[(int64_t)m * p.N + n] = sC[row * LDC + col];
            }
        }
        return;
    }
    if constexpr (MODE == STORE_ANY) {
        if constexpr (AHEAD) if (pe.form != PE_NONE) {
            // two passes of 32 rows at a time, one in stage 0's array and one in stage 1's
            static_assert(32 * (BN + 1) * 4 <= STAGE, "a pass must fit in one stage");
            float *sD = (float *)st1;
#pragma unroll
            for (int q = 0; q < BM / 32; q += 2) {
                wg_barrier();                       // previous passes read out / last K tile consumed
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int own = wm * TM + i;
                    if (own >> 1 == q >> 1) {
                        float *dst = own & 1 ? sD : sC;
#pragma unroll
                        for (int j = 0; j < TN; ++j)
#pragma unroll
                            for (int r = 0; r < 16; ++r) {
                                int row = 8 * (r >> 2) + 4 * fhalf + (r & 3);
                                int col = wn * WTN + j * 32 + frow;
                                dst[row * (BN + 1) + col] = acc[i][j][r];
                            }
                    }
                }
                __syncthreads();
                pe.store(p, sC, t, m0, n0, q);
                pe.store(p, sD, t, m0, n0, q + 1);
            }
            return;
        }
        // the loop stays rolled (its pass inlined BM / 32 times costs the registers of a second workgroup per CU), rows BN + 1
        // floats apart for the reads down a column
#pragma unroll 1
        for (int q = 0; q < BM / 32; ++q) {
            wg_barrier();                           // previous pass read out / last K tile consumed
            if (wm == q / TM) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    if (i == q % TM) {
#pragma unroll
                        for (int j = 0; j < TN; ++j)
#pragma unroll
                            for (int r = 0; r < 16; ++r) {
                                int row = 8 * (r >> 2) + 4 * fhalf + (r & 3);
                                int col = wn * WTN + j * 32 + frow;
                                sC[row * (BN + 1) + col] = acc[i][j][r];
                            }
                    }
            }
            __syncthreads();
            TE::store_pass_scalar(p, sC, BN + 1, t, m0 + q * 32, n0);
        }
        return;
    }
    if constexpr (TEAMS == 1) request_rows();
#pragma unroll
    for (int q = 0; q < BM / 32; ++q) {
        if (pre && q + 1 < BM / 32) TE::prefetch(p, t, m0 + (q + 1) * 32, n0, nxt);
        wg_barrier();                           // previous pass read out / last K tile consumed
        if (wm == q / TM) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    int row = 8 * (r >> 2) + 4 * fhalf + (r & 3);
                    int col = wn * WTN + j * 32 + frow;
                    sC[row * LDC + col] = acc[q % TM][j][r];
                }
        }
        __syncthreads();
        const int mq = m0 + q * 32;
        if (GATES) TE::gates_pass(p, sC, LDC, t, mq, bn);
        else TE::store_pass(p, sC, LDC, t, mq, n0, bias8, cur);
        cur = nxt;
    }
#endif
}

}  // namespace rl
