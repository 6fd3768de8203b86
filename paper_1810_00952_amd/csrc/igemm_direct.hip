// Contractions too small to fill the chip with LDS tiles: operands go from memory straight into MFMA registers, and K is cut over
// the waves of a workgroup, whose sums meet in LDS.
//
//   C[m, n] = sum_k A[m, k] * Wp[n, k], then the group's epilogue, any result strides, and a 2x2 / stride 2 max-pool if one follows
//
// What bounds these calls is launches and latencies, not work: cut over workgroups the sums meet in a scratch tensor that a second
// launch adds up, and a channel-first operand is copied first.  Here the whole call is one launch: a wave has eight K steps of both
// operands in flight, the slices meet behind one barrier, and the operands of the epilogue are requested ahead of the products.
// One image of 64x56x56 through 3x3 to 64 channels, f32: 17.5 us (copy, split contraction, adding launch) -> 8.8; LeNet's shape,
// batch 64, 62 -> 28 (its max-pools and a change of layout ride along).
// No LDS tile: a lane of an MFMA operand needs 16 bytes of its own row, and neighbouring lanes' rows lie apart, so that a load of 1 KB
// occupies the vector L1 for about 50 cycles (8 waves' step 780 cycles on a CU, its f32 MFMAs 512).  That is what sends
// larger contractions to the kernels with LDS tiles; Planner::direct_form has the line.
// A convolution's weights that it alone reads are packed in the order of its fragments (pack_weight_direct_kernel), a load then being a
// KB in a row: 64x56x56 -> 64 3x3 f32 8.77 -> 8.13 us; other small layers 1.00 to 1.02 of their rate before, none slower.
// 32x32 tiles, or 16x16 with eight slices where there are few: half the K steps per wave and four times the workgroups.
#include <algorithm>

#include "igemm_epilogue.h"
#include "igemm_lds.h"

namespace rl {

namespace {

constexpr int WAVES = 8;

template <int TS> struct Acc { f32x16 v; };
template <> struct Acc<16> { f32x4 v; };

// one 16-byte chunk of K per lane on either side: f32 four MFMAs, lane group g supplying k = 4 g + j to the j-th; bf16 one
template <typename T, int TS> __device__ __forceinline__ void mma(Acc<TS> &acc, const u32x4 &a, const u32x4 &b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (TS == 32) acc.v = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[j]), __uint_as_float(b[j]), acc.v, 0, 0, 0);
            else acc.v = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[j]), __uint_as_float(b[j]), acc.v, 0, 0, 0);
        }
    } else {
        if constexpr (TS == 32) acc.v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc.v, 0, 0, 0);
        else acc.v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc.v, 0, 0, 0);
    }
#endif
}

}  // namespace

// MODE: how a lane gets its chunk of A (16 bytes of consecutive k = (tap, channel)).
//   ROWS    channels fastest in memory and whole chunks of them: one 16-byte load
//   PLANES  whole chunks of channels, any strides: one load per channel, neighbouring lanes neighbouring pixels
//   ANY     every element decoded by itself
// WB: the weights lie in rows of K (W_ROWS), in the order of the fragments (W_FRAGMENTS), or in rows of N, of which a lane takes its column
// element by element (W_COLUMNS: x of a dense weight gradient)
enum { W_ROWS = 0, W_FRAGMENTS = 1, W_COLUMNS = 2 };
template <typename T, int MODE, int TS, int KS, int WB>
__global__ __launch_bounds__(64 * WAVES) void igemm_direct_kernel(const IgemmParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub; the body uses gfx950-only builtins
    constexpr int KV = Elem<T>::KV, ES = (int)sizeof(T);
    constexpr int G = 64 / TS;                       // lane groups: chunks of K per step
    constexpr int WT = WAVES / KS, BM = WT * TS;     // tiles (of TS x TS) per workgroup, one under the other
    constexpr int LD = TS + 1;
    constexpr int AV = MODE == DIRECT_ROWS ? 4 : KV; // registers of a chunk of A in flight
    constexpr int BV = WB == W_COLUMNS ? KV : 4;     // ... and of the weights
    constexpr int DEPTH = AV == 8 || BV == 8 ? 4 : 8; // steps in flight
    constexpr int PER = TS * TS * WT / (64 * WAVES); // results per thread (0: half of the threads have one)
    constexpr int EPT = PER < 1 ? 1 : PER;
    __shared__ float part[WAVES][TS * LD];

    touch_args(p);
    // what the first request hangs on
    asm volatile("" :: "s"(p.nblk_m), "s"(p.nblk_n), "s"(p.x), "s"(p.w), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.Kp), "s"(p.C), "s"(p.H), "s"(p.W), "s"(p.KH), "s"(p.KW), "s"(p.OW), "s"(p.OHW), "s"(p.sh), "s"(p.sw),
                 "s"(p.ph), "s"(p.pw), "s"(p.xs_n), "s"(p.xs_c), "s"(p.xs_h), "s"(p.xs_w), "s"(p.x_bytes), "s"(p.w_bytes), "s"(p.pool));
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int slice = wave % KS, tw = wave / KS;
    const int bid = xcd_run(blockIdx.x, p.nblk_m * p.nblk_n);
    const int bm = bid / p.nblk_n, bn = bid - bm * p.nblk_n;
    const int m0 = bm * BM, n0 = bn * TS;
    const int l = lane % TS, g = lane / TS;

    const rsrc_t rx = make_rsrc(p.x, p.x_bytes);
    const rsrc_t rw = make_rsrc(p.w, p.w_bytes);
    auto div_ohw = [&](int v) { return p.OHW == 1 ? v : (int)(__umulhi((uint32_t)v, p.div_ohw_mul) >> p.div_ohw_sh); };
    auto div_ow = [&](int v) { return p.OW == 1 ? v : (int)(__umulhi((uint32_t)v, p.div_ow_mul) >> p.div_ow_sh); };
    auto div_c = [&](int v) { return p.C == 1 ? v : (int)(__umulhi((uint32_t)v, p.div_c_mul) >> p.div_c_sh); };
    auto div_kw = [&](int v) { return p.KW == 1 ? v : (int)(__umulhi((uint32_t)v, p.div_kw_mul) >> p.div_kw_sh); };

    // ---- the lane's row of A and of the weights
    const bool one_tap = p.KH * p.KW == 1;
    int ih0, iw0;
    uint32_t a_off;                                  // of tap (0, 0): may lie before x, the taps inside the image never do
    {
        const int m = m0 + tw * TS + l;
        const int q = p.pool ? m >> 2 : m, d = p.pool ? m & 3 : 0;       // with a pool the four pixels of a window follow one another
        const int img = div_ohw(q), pix = q - img * p.OHW;
        const int qh = div_ow(pix), qw = pix - qh * p.OW;
        const int oh = p.pool ? 2 * qh + (d >> 1) : qh, ow = p.pool ? 2 * qw + (d & 1) : qw;
        ih0 = m < p.M ? oh * p.sh - p.ph : -(1 << 24);
        iw0 = ow * p.sw - p.pw;
        a_off = (uint32_t)(((int64_t)img * p.xs_n + (int64_t)(oh * p.sh - p.ph) * p.xs_h + (int64_t)iw0 * p.xs_w) * ES);
    }
    const int n = n0 + l;
    const uint32_t b_off = (uint32_t)((int64_t)n * p.Kp * ES);
    const bool n_live = n < p.N;
    const bool row_live = (unsigned)ih0 < (unsigned)p.H && (unsigned)iw0 < (unsigned)p.W;
    const uint32_t xs_c = (uint32_t)(p.xs_c * ES), xs_h = (uint32_t)(p.xs_h * ES), xs_w = (uint32_t)(p.xs_w * ES);

    const int S = (p.K + KV * G - 1) / (KV * G);
    const int s0 = slice * S / KS, s1 = (slice + 1) * S / KS;
    uint32_t fa[DEPTH][AV];
    uint32_t fb[DEPTH][BV];
    // offset of element k, or out of range: padding, rows past M, k past K
    auto a_at = [&](int k) -> uint32_t {
        if (one_tap) return row_live && k < p.K ? a_off + (uint32_t)k * xs_c : OOB;
        const int tap = div_c(k), c = k - tap * p.C, kh = div_kw(tap), kw = tap - kh * p.KW;
        const bool ok = (unsigned)(ih0 + kh) < (unsigned)p.H && (unsigned)(iw0 + kw) < (unsigned)p.W && k < p.K;
        return ok ? a_off + (uint32_t)kh * xs_h + (uint32_t)kw * xs_w + (uint32_t)c * xs_c : OOB;
    };
    auto load1 = [&](uint32_t off) -> uint32_t {
        if constexpr (ES == 4) return __builtin_amdgcn_raw_buffer_load_b32(rx, off, 0, 0);
        else return __builtin_amdgcn_raw_buffer_load_b16(rx, off, 0, 0);
    };
    auto fetch = [&](int slot, int step) {
        const int k = (step * G + g) * KV;
        if constexpr (WB == W_COLUMNS) {
#pragma unroll
            for (int e = 0; e < KV; ++e) {
                const uint32_t off = n_live && k + e < p.K ? (uint32_t)((k + e) * p.Kp + n) * ES : OOB;
                if constexpr (ES == 4) fb[slot][e] = __builtin_amdgcn_raw_buffer_load_b32(rw, off, 0, 0);
                else fb[slot][e] = __builtin_amdgcn_raw_buffer_load_b16(rw, off, 0, 0);
            }
        } else {
            constexpr bool FRAG = WB == W_FRAGMENTS;
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rw, FRAG ? (uint32_t)lane * 16u : n_live && k < p.Kp ? b_off + (uint32_t)(k * ES) : OOB, FRAG ? (uint32_t)(bn * S + step) * 1024u : 0u, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) fb[slot][e] = v[e];
        }
        if constexpr (MODE == DIRECT_ANY) {
#pragma unroll
            for (int e = 0; e < KV; ++e) fa[slot][e] = load1(a_at(k + e));
        } else {
            const uint32_t off = a_at(k);
            if constexpr (MODE == DIRECT_ROWS) {
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) fa[slot][e] = v[e];
            } else {
#pragma unroll
                for (int e = 0; e < KV; ++e) fa[slot][e] = load1(off == OOB ? OOB : off + (uint32_t)e * xs_c);
            }
        }
    };
    auto chunk = [](const auto &f) -> u32x4 {
        u32x4 v;
        if constexpr (sizeof(f) == 16) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = f[e];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = f[2 * e] | (f[2 * e + 1] << 16);
        }
        return v;
    };
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
        if (s0 + i < s1) fetch(i, s0 + i);           // (the wave's last steps take their chunks' addresses for nothing otherwise: most of a short K's time)
    __builtin_amdgcn_sched_barrier(0);               // all of them in flight before the first is used

    // ---- the results this thread finishes: lanes along the result's fastest axis, and along the other one a fixed step apart, so
    // that one of row and column stays the same for all of them
    const Epilogue &e = p.epi;
    const bool pix_fast = p.ys_p == 1 && p.OHW > 1;
    const int ys_n = (int)p.ys_n, ys_p = (int)p.ys_p, ys_c = (int)p.ys_c;      // the result has fewer than 2^31 elements
    const bool even = ys_n == p.OHW * ys_p;          // images follow one another like pixels
    auto y_row = [&](int m) -> int {                 // m: (pooled) pixel
        if (even) return m * ys_p;
        const int img = div_ohw(m);
        return img * ys_n + (m - img * p.OHW) * ys_p;
    };
    constexpr int ML_STEP = 64 * WAVES / TS, COL_STEP = 64 * WAVES / BM > 0 ? 64 * WAVES / BM : 1;
    const int ml0 = pix_fast ? t % BM : t / TS, col0 = pix_fast ? t / BM : t % TS;
    auto ml_of = [&](int i) { return pix_fast ? ml0 : ml0 + ML_STEP * i; };
    auto col_of = [&](int i) { return pix_fast ? col0 + COL_STEP * i : col0; };
    constexpr int CH = EPT < 4 ? EPT : 4;            // results at a time; the operands of the first ones are requested ahead of the products
    float bias[CH], tt[CH];
    int off[CH];
    const int base = pix_fast ? y_row(m0 + ml0) : (n0 + col0) * ys_c;
    auto operands = [&](int i0) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int m = m0 + ml_of(i0 + i), nn = n0 + col_of(i0 + i);
            const bool live = (PER >= 1 || t < TS * TS * WT) && m < p.M && nn < p.N;
            off[i] = live ? base + (pix_fast ? nn * ys_c : y_row(m)) : -1;
            bias[i] = live && e.simple && e.has_bias ? load_as_f32(e.bias_ptr, e.bias_dtype, nn) : 0.0f;
            tt[i] = live && e.simple && e.t_op >= 0 ? load_as_f32(e.t_ptr, e.t_dtype, off[i]) : 0.0f;
        }
    };
    if (!p.pool) {
        operands(0);
        __builtin_amdgcn_sched_barrier(0);
    }

    Acc<TS> acc;
#pragma unroll
    for (int i = 0; i < TS * TS / 64; ++i) acc.v[i] = 0.0f;
    const int steps = s1 - s0;
#pragma unroll 1
    for (int b = 0; b < steps; b += DEPTH) {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) {
            if (b + i >= steps) break;
            mma<T, TS>(acc, chunk(fa[i]), chunk(fb[i]));
            if (b + i + DEPTH < steps) fetch(i, s0 + b + i + DEPTH);
        }
    }
#pragma unroll
    for (int r = 0; r < TS * TS / 64; ++r) {
        const int row = TS == 32 ? 8 * (r >> 2) + 4 * g + (r & 3) : 4 * g + r;
        part[wave][row * LD + l] = acc.v[r];
    }
    __syncthreads();

    auto sum = [&](int ml, int col) {                // slices in order
        const int w0 = ml / TS * KS, q = (ml % TS) * LD + col;
        float v = part[w0][q];
#pragma unroll
        for (int s = 1; s < KS; ++s) v += part[w0 + s][q];
        return v;
    };
    if (!p.pool) {
#pragma unroll 1
        for (int i0 = 0; i0 < EPT; i0 += CH) {
            if (i0 > 0) operands(i0);
            float v[CH];
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                v[i] = sum(ml_of(i0 + i) % BM, col_of(i0 + i) % TS);     // (fewer results than threads: those of the others are not used)
                if (!e.simple && off[i] >= 0)
                    for (int s = 0; s < e.n_ops; ++s) v[i] = epi_step(e, s, v[i], off[i], n0 + col_of(i0 + i));
            }
            if (e.simple) TileEpilogue<64>::template finish<CH>(e, v, bias, tt);
#pragma unroll
            for (int i = 0; i < CH; ++i)
                if (off[i] >= 0) store_from_f32(p.y, p.y_dtype, off[i], v[i]);
        }
        return;
    }
    // a 2x2 window per result: every value finished and rounded as the tensor between the two groups would hold it, then the largest
    constexpr int WIN = BM / 4 * TS;
#pragma unroll 1
    for (int idx = t; idx < WIN; idx += 64 * WAVES) {
        int wl, col;
        if (pix_fast) { wl = idx % (BM / 4); col = idx / (BM / 4); }
        else { col = idx % TS; wl = idx / TS; }
        const int m = m0 / 4 + wl, nn = n0 + col;
        if (4 * m >= p.M || nn >= p.N) continue;
        float v[4], bs[4], zero[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        const float b = e.has_bias ? load_as_f32(e.bias_ptr, e.bias_dtype, nn) : 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) { v[k] = sum(4 * wl + k, col); bs[k] = b; }
        TileEpilogue<64>::template finish<4>(e, v, bs, zero);
        float best = -INFINITY;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float r = p.y_dtype == DT_BF16 ? round_bf16(v[k]) : v[k];
            best = r > best ? r : best;
        }
        store_from_f32(p.y, p.y_dtype, y_row(m) + nn * ys_c, best);
    }
#endif
}

// A recurrent cell: z = [x, h] Wp^T (packed rows: 64 = 4 gates x 16 units of a block), then the bias and the gates.
// A workgroup has 16 batch rows and UN units, all four gates of them; its waves take a slice of K each, so that every memory latency
// of the step is paid once.  What bounds a step behind that and its launch is the vector L1's 50 cycles per load of a fragment, on
// however many CUs take part: few units per workgroup where there are few rows.
// 160 drawn sequences: f32 0.25 of the time, bf16 0.22, none above 0.80 (us a step: f32 42 rows, 928 -> 544 units 34 -> 17; 12 rows, 96 -> 48, bf16 12.6 -> 3.6).
// (The element gather, which ran wherever the width of x or h was no multiple of the K tile, read one element at a time on one workgroup
// per 64 rows and block.)
template <typename T, int UN>
__global__ __launch_bounds__(64 * WAVES) void lstm_cell_direct_kernel(const IgemmParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int KV = Elem<T>::KV, ES = (int)sizeof(T);
    constexpr int TS = 16, G = 64 / TS, NT = UN / 4; // column tile j: units 4 j .. 4 j + 3, column 4 gate + unit
    constexpr int LD = TS + 1, DEPTH = 4;
    constexpr int PAIRS = TS * UN;                   // (row, unit) pairs, one per thread
    __shared__ float part[WAVES][NT][TS * LD];

    touch_args(p);
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int unit0 = blockIdx.x * UN, m0 = blockIdx.y * TS;
    const int l = lane % TS, g = lane / TS;

    // ---- what the thread finishes
    const Epilogue &e = p.epi;
    const int prow = t / UN, pu = t % UN, pm = m0 + prow, unit = unit0 + pu;
    const bool fin = t < PAIRS && pm < p.M;
    const int64_t at = (int64_t)pm * p.hidden + unit;
    float bias[4] = {0.0f, 0.0f, 0.0f, 0.0f}, c = 0.0f;
    if (fin) {
        c = p.c_in[at];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (e.n_ops == 1) bias[q] = load_as_f32(e.bias_ptr, e.bias_dtype, q * p.hidden + unit);
    }

    const rsrc_t rx = make_rsrc(p.x, p.x_bytes), rh = make_rsrc(p.x2, p.x2_bytes), rw = make_rsrc(p.w, p.w_bytes);
    const int m = m0 + l;
    const uint32_t x_off = (uint32_t)((int64_t)m * p.xs_n * ES), h_off = (uint32_t)((int64_t)m * p.x2s_n * ES);
    const uint32_t w_off = (uint32_t)((int64_t)((unit0 >> 4) * 64 + (l >> 2) * 16 + (unit0 & 15) + (l & 3)) * p.Kp * ES), w_tile = (uint32_t)((int64_t)4 * p.Kp * ES);
    const int S = (p.K + KV * G - 1) / (KV * G);
    const int s0 = wave * S / WAVES, s1 = (wave + 1) * S / WAVES, steps = s1 - s0;
    u32x4 fx[DEPTH], fh[DEPTH], fb[DEPTH][NT];
    auto fetch = [&](int slot, int step) {
        const int k = (step * G + g) * KV;
        const bool live = m < p.M && k < p.K, first = k < p.K1;
        // of the two operands' loads one is out of range and reads as zero
        fx[slot] = __builtin_amdgcn_raw_buffer_load_b128(rx, live && first ? x_off + (uint32_t)(k * ES) : OOB, 0, 0);
        fh[slot] = __builtin_amdgcn_raw_buffer_load_b128(rh, live && !first ? h_off + (uint32_t)((k - p.K1) * ES) : OOB, 0, 0);
#pragma unroll
        for (int j = 0; j < NT; ++j) fb[slot][j] = __builtin_amdgcn_raw_buffer_load_b128(rw, k < p.Kp ? w_off + (uint32_t)j * w_tile + (uint32_t)(k * ES) : OOB, 0, 0);
    };
    Acc<TS> acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < TS * TS / 64; ++i) acc[j].v[i] = 0.0f;
#pragma unroll 1
    for (int b = 0; b < steps; b += DEPTH) {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i)
            if (b + i < steps) fetch(i, s0 + b + i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) {
            if (b + i >= steps) break;
#pragma unroll
            for (int j = 0; j < NT; ++j) mma<T, TS>(acc[j], fx[i] | fh[i], fb[i][j]);
        }
    }
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < TS * TS / 64; ++r) part[wave][j][(4 * g + r) * LD + l] = acc[j].v[r];
    __syncthreads();
    if (!fin) return;
    float z[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float v = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) v += part[w][pu >> 2][prow * LD + 4 * q + (pu & 3)];
        z[q] = v + bias[q];
    }
    const float hn = lstm_cell_(z, c);
    p.c_out[at] = c;
    store_from_f32(p.h_out, p.h_dtype, at, hn);
#endif
}
#define RL_INST(UN) template __global__ void lstm_cell_direct_kernel<float, UN>(const IgemmParams); template __global__ void lstm_cell_direct_kernel<uint16_t, UN>(const IgemmParams);
RL_INST(4) RL_INST(8)
#undef RL_INST

#define RL_ONE(T, MODE, TS, KS, WB) template __global__ void igemm_direct_kernel<T, MODE, TS, KS, WB>(const IgemmParams);
#define RL_FIVE(T, MODE, WB) RL_ONE(T, MODE, 32, 1, WB) RL_ONE(T, MODE, 32, 2, WB) RL_ONE(T, MODE, 32, 4, WB) RL_ONE(T, MODE, 32, 8, WB) RL_ONE(T, MODE, 16, 8, WB)
#define RL_INST(T, MODE) RL_FIVE(T, MODE, W_ROWS) RL_FIVE(T, MODE, W_FRAGMENTS)
RL_INST(float, DIRECT_ROWS) RL_INST(float, DIRECT_PLANES) RL_INST(float, DIRECT_ANY)
RL_INST(uint16_t, DIRECT_ROWS) RL_INST(uint16_t, DIRECT_PLANES) RL_INST(uint16_t, DIRECT_ANY)
RL_FIVE(float, DIRECT_ANY, W_COLUMNS) RL_FIVE(uint16_t, DIRECT_ANY, W_COLUMNS)
#undef RL_FIVE
#undef RL_ONE
#undef RL_INST

template <typename T, int MODE, int TS, int KS>
static hipError_t launch_one(const IgemmParams &p0, hipStream_t s)
{
    IgemmParams p = p0;
    constexpr int BM = WAVES / KS * TS;
    p.nblk_m = (p.M + BM - 1) / BM;
    p.nblk_n = (p.N + TS - 1) / TS;
    const int64_t nblk = (int64_t)p.nblk_m * p.nblk_n;
    if (nblk <= 0 || nblk > 0x7fffffff) return hipErrorInvalidValue;
    if (p.w_frag == W_COLUMNS) {
        if constexpr (MODE == DIRECT_ANY) hipLaunchKernelGGL((igemm_direct_kernel<T, MODE, TS, KS, W_COLUMNS>), dim3((unsigned)nblk), dim3(64 * WAVES), 0, s, p);
        else return hipErrorInvalidValue;
    } else if (p.w_frag) hipLaunchKernelGGL((igemm_direct_kernel<T, MODE, TS, KS, W_FRAGMENTS>), dim3((unsigned)nblk), dim3(64 * WAVES), 0, s, p);
    else hipLaunchKernelGGL((igemm_direct_kernel<T, MODE, TS, KS, W_ROWS>), dim3((unsigned)nblk), dim3(64 * WAVES), 0, s, p);
    return hipGetLastError();
}

template <typename T, int MODE> static hipError_t launch_mode(const IgemmParams &p, const IgemmLaunch &l, hipStream_t s)
{
    if (l.direct_tile == 16) return launch_one<T, MODE, 16, 8>(p, s);
    switch (l.direct_slices) {
    case 1: return launch_one<T, MODE, 32, 1>(p, s);
    case 2: return launch_one<T, MODE, 32, 2>(p, s);
    case 4: return launch_one<T, MODE, 32, 4>(p, s);
    default: return launch_one<T, MODE, 32, 8>(p, s);
    }
}

template <typename T> static hipError_t launch_typed(const IgemmParams &p, const IgemmLaunch &l, hipStream_t s)
{
    switch (l.direct - 1) {
    case DIRECT_ROWS: return launch_mode<T, DIRECT_ROWS>(p, l, s);
    case DIRECT_PLANES: return launch_mode<T, DIRECT_PLANES>(p, l, s);
    default: return launch_mode<T, DIRECT_ANY>(p, l, s);
    }
}

template <int UN> static void launch_cell(const IgemmParams &p, hipStream_t s)
{
    const dim3 grid((unsigned)(p.hidden / UN), (unsigned)((p.M + 15) / 16));
    if (p.in_dtype == DT_BF16) hipLaunchKernelGGL((lstm_cell_direct_kernel<uint16_t, UN>), grid, dim3(64 * WAVES), 0, s, p);
    else hipLaunchKernelGGL((lstm_cell_direct_kernel<float, UN>), grid, dim3(64 * WAVES), 0, s, p);
}

static hipError_t launch_lstm_cell(const IgemmParams &p, int units, hipStream_t s)
{
    const int KV = p.in_dtype == DT_BF16 ? 8 : 4, ES = 16 / KV;
    const int64_t K2 = p.K - p.K1;
    if (!p.x || !p.x2 || !p.w || !p.c_in || !p.c_out || !p.h_out || p.M < 1 || p.M > 65535 * 16 || p.K1 < 1 || K2 < 1 || p.K1 % KV || K2 % KV || p.xs_n % KV || p.x2s_n % KV || p.Kp < p.K || p.Kp % KV ||
        p.hidden % 16 || p.N != 4 * p.hidden || (p.epi.n_ops > 1) || (p.epi.n_ops == 1 && !p.epi.has_bias) || (uint64_t)p.N * p.Kp * ES > p.w_bytes ||
        (uint64_t)((p.M - 1) * p.xs_n + p.K1) * ES > p.x_bytes || (uint64_t)((p.M - 1) * p.x2s_n + K2) * ES > p.x2_bytes || p.x_bytes >= OOB || p.x2_bytes >= OOB || p.w_bytes >= OOB)
        return hipErrorInvalidValue;
    if (units == 4) launch_cell<4>(p, s);
    else launch_cell<8>(p, s);
    return hipGetLastError();
}

hipError_t launch_igemm_direct(const IgemmParams &p, const IgemmLaunch &l, hipStream_t s)
{
    const int KV = p.in_dtype == DT_BF16 ? 8 : 4;
    if (l.gates) return launch_lstm_cell(p, l.direct_units, s);
    if (!p.x || !p.w || !p.y || p.x2 || p.M < 1 || p.N < 1 || p.K < 1 || p.K != p.C * p.KH * p.KW || p.x_bytes >= OOB || p.w_bytes >= OOB ||
        (p.w_frag == W_COLUMNS ? p.Kp < p.N || p.KH * p.KW != 1 || (uint64_t)p.K * p.Kp * (16 / KV) > p.w_bytes : p.Kp < p.K || p.Kp % KV != 0 || (uint64_t)p.N * p.Kp * (16 / KV) > p.w_bytes) ||
        (p.w_frag == W_FRAGMENTS && (p.Kp != (p.K + KV * (64 / l.direct_tile) - 1) / (KV * (64 / l.direct_tile)) * KV * (64 / l.direct_tile) ||
        (uint64_t)((p.N + l.direct_tile - 1) / l.direct_tile * l.direct_tile) * p.Kp * (16 / KV) > p.w_bytes)) || (l.direct - 1 != DIRECT_ANY && p.C % KV != 0) || (l.direct - 1 == DIRECT_ROWS && p.xs_c != 1) ||
        (int64_t)p.M * p.N >= (int64_t)1 << 31 || (p.pool && (!p.epi.simple || p.epi.t_op >= 0 || p.M % 4 != 0)) || p.tap_dil_m1 || p.in_dil_m1)
        return hipErrorInvalidValue;
    return p.in_dtype == DT_BF16 ? launch_typed<uint16_t>(p, l, s) : launch_typed<float>(p, l, s);
}

}  // namespace rl
