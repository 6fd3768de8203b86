// Epilogue of the contraction kernels: 32 rows of fp32 accumulators staged in
// LDS (row stride LDC floats) are turned into output rows, 8 consecutive
// channels per thread, with the group's injective chain applied in between.
//
// A thread keeps the same 8 channels for every row it touches, so a leading
// bias_add is loaded once, and the one full-shape operand most chains have
// (the residual) is fetched one 32-row pass ahead: global-load latency is paid
// once per tile instead of once per dependent step.  Chains of another form
// take the generic path (operands loaded where the chain needs them).
#pragma once
#include "device_utils.h"

namespace rl {

// The chain's form is classified on the host (Epilogue::simple, has_bias, t_op, rest_ops and the
// resolved bias_ptr / t_ptr), so the kernels read fixed kernel-argument fields here.
// One thread's operand vectors for one 32-row pass (raw 16 or 32 bytes each).
template <int NV> struct OperandRegs { u32x4 lo[NV], hi[NV]; };

template <int BN>
struct TileEpilogue {
    static constexpr int VPR = BN / 8;            // 8-channel vectors per row
    static constexpr int SWEEP = 256 / VPR;       // rows covered by the 256 threads at once
    static constexpr int NV = 32 / SWEEP;         // vectors per thread per 32-row pass

    // issue the loads of the full-shape operand for the rows of one pass
    static __device__ __forceinline__ void prefetch(const IgemmParams &p, int t, int mq, int n0,
                                                    OperandRegs<NV> &r)
    {
        const int cv = t % VPR, r0 = t / VPR;
        const int n = n0 + cv * 8;
        const void *ptr = p.epi.t_ptr;
        const bool f32 = p.epi.t_dtype == DT_F32;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int m = mq + r0 + SWEEP * i;
            r.lo[i] = u32x4{0u, 0u, 0u, 0u};
            r.hi[i] = u32x4{0u, 0u, 0u, 0u};
            if (p.epi.t_op >= 0 && m < p.M && n < p.N) {
                const int64_t off = (int64_t)m * p.ys_p + n;
                if (f32) {
                    r.lo[i] = *(const u32x4 *)((const float *)ptr + off);
                    r.hi[i] = *(const u32x4 *)((const float *)ptr + off + 4);
                } else {
                    r.lo[i] = *(const u32x4 *)((const uint16_t *)ptr + off);
                }
            }
        }
    }

    static __device__ __forceinline__ void load_bias(const IgemmParams &p, int t, int n0, float b[8])
    {
        const int n = n0 + (t % VPR) * 8;
#pragma unroll
        for (int k = 0; k < 8; ++k) b[k] = 0.0f;
        if (p.epi.has_bias && n < p.N) load8(p.epi.bias_ptr, p.epi.bias_dtype, n, b);
    }

    // rows mq .. mq+31 from sC; output row-major with 8 | N (checked by the caller)
    static __device__ __forceinline__ void store_pass(const IgemmParams &p, const float *sC, int ldc, int t,
                                                      int mq, int n0, const float bias[8], const OperandRegs<NV> &r)
    {
        const Epilogue &e = p.epi;
        const int cv = t % VPR, r0 = t / VPR;
        const int n = n0 + cv * 8;
        const bool f32 = e.t_op >= 0 && e.t_dtype == DT_F32;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int row = r0 + SWEEP * i;
            const int m = mq + row;
            if (m < p.M && n < p.N) {
                float val[8];
                f32x4 lo = *(const f32x4 *)(sC + row * ldc + cv * 8);
                f32x4 hi = *(const f32x4 *)(sC + row * ldc + cv * 8 + 4);
#pragma unroll
                for (int k = 0; k < 4; ++k) { val[k] = lo[k]; val[4 + k] = hi[k]; }
                const int64_t off = (int64_t)m * p.ys_p + n;
                if (e.simple) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) val[k] += bias[k];
                    if (e.t_op >= 0) {
                        float tt[8];
                        if (f32) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) { tt[k] = __uint_as_float(r.lo[i][k]); tt[4 + k] = __uint_as_float(r.hi[i][k]); }
                        } else {
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                tt[2 * k] = __uint_as_float(r.lo[i][k] << 16);
                                tt[2 * k + 1] = __uint_as_float(r.lo[i][k] & 0xffff0000u);
                            }
                        }
#pragma unroll
                        for (int k = 0; k < 8; ++k) val[k] = binop(e.t_op, val[k], tt[k]);
                    }
                    uint64_t codes = e.rest_ops;
                    for (int s = 0; s < e.rest_n; ++s, codes >>= 8) {
                        const int op = (int)(codes & 0xff);
                        if (op == E_RELU) {
#pragma unroll
                            for (int k = 0; k < 8; ++k) val[k] = val[k] > 0.0f ? val[k] : 0.0f;
                        } else {
#pragma unroll
                            for (int k = 0; k < 8; ++k) val[k] = unary_step(op, val[k]);
                        }
                    }
                } else {
                    chain8(e, val, off, n, 1, p.N);
                }
                store8(p.y, p.y_dtype, off, val);
            }
        }
    }

    // K values through a simple chain (one switch per step, not per value)
    template <int K> static __device__ __forceinline__ void finish(const Epilogue &e, float (&val)[K], const float (&bias)[K], const float (&tt)[K])
    {
#pragma unroll
        for (int k = 0; k < K; ++k) val[k] += bias[k];
        if (e.t_op >= 0) {
#pragma unroll
            for (int k = 0; k < K; ++k) val[k] = binop(e.t_op, val[k], tt[k]);
        }
        uint64_t codes = e.rest_ops;
        for (int s = 0; s < e.rest_n; ++s, codes >>= 8) {
            const int op = (int)(codes & 0xff);
            if (op == E_RELU) {
#pragma unroll
                for (int k = 0; k < K; ++k) val[k] = val[k] > 0.0f ? val[k] : 0.0f;
            } else {
#pragma unroll
                for (int k = 0; k < K; ++k) val[k] = unary_step(op, val[k]);
            }
        }
    }

    // Results in Shape order (channel-first) and ragged N.  What bounds this pass is how its stores and operand loads
    // coalesce, and the index arithmetic: an element at a time with two divisions and the interpreted chain each took most of
    // a 77 us convolution (17x96x29x29 -> 136, bf16, residual).  A thread keeps its pixels for the pass (decoded once, by
    // multiply-high) and walks channels, operands requested a few channels at a time: four pixels of one channel as one store
    // where images are whole groups of four pixels, one pixel otherwise; results with channels fastest go element by
    // element across lanes.  sC rows are ldc floats apart: BN + 1 spreads the columns read here over the banks.
    // (Loops are kept rolled: the pass inlined once per 32 rows took 230 VGPRs and one wave per SIMD.)
    static __device__ __forceinline__ void store_pass_scalar(const IgemmParams &p, const float *sC, int ldc, int t, int mq, int n0)
    {
        const Epilogue &e = p.epi;
        const bool tload = e.t_op >= 0;
        const bool chan_fast = p.ys_c == 1;
        const bool even_rows = p.ys_n == (int64_t)p.OHW * p.ys_p;        // images follow one another like pixels
        auto row_off = [&](int m) -> int64_t {
            if (even_rows) return (int64_t)m * p.ys_p;
            const int img = p.OHW == 1 ? m : (int)(__umulhi((uint32_t)m, p.div_ohw_mul) >> p.div_ohw_sh);
            return (int64_t)img * p.ys_n + (int64_t)(m - img * p.OHW) * p.ys_p;
        };
        if (e.simple && chan_fast && p.N - n0 >= BN) {
            // channels fastest, N no multiple of eight, a whole tile of channels: a thread keeps its channel, four rows at a time
            constexpr int RS = 256 / BN;
            const int col = t % BN, n = n0 + col;
            const float b = e.has_bias ? load_as_f32(e.bias_ptr, e.bias_dtype, n) : 0.0f;
#pragma unroll 1
            for (int r0 = t / BN; r0 < 32; r0 += 4 * RS) {
                float v[4], bias[4], tt[4];
                int64_t off[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int m = mq + r0 + RS * i;
                    off[i] = row_off(m) + n;
                    v[i] = sC[(r0 + RS * i) * ldc + col];
                    bias[i] = b;
                    tt[i] = tload && m < p.M ? load_as_f32(e.t_ptr, e.t_dtype, off[i]) : 0.0f;
                }
                finish<4>(e, v, bias, tt);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (mq + r0 + RS * i < p.M) store_from_f32(p.y, p.y_dtype, off[i], v[i]);
            }
            return;
        }
        if (e.simple && chan_fast) {
            // the last, partial tile of channels: the pass's elements one after the other over all threads, four of them at a time
            // each, so that few channels leave no thread idle while another has several rows to go (dense 704 x 208 -> 4 bf16: a
            // channel per thread 9.1 us, this 6.1; 14 x 240 -> 1697 on whole tiles 6.9 against 7.5)
            const int cols = p.N - n0, total = 32 * cols;
            const uint32_t inv = (1u << 20) / (uint32_t)cols + 1u;            // idx / cols: exact below 2^20 / 128
#pragma unroll 1
            for (int i0 = t; i0 < total; i0 += 1024) {
                float v[4], bias[4], tt[4];
                int64_t off[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int idx = i0 + 256 * i, row = (int)(((uint32_t)idx * inv) >> 20), col = idx - row * cols;
                    const int m = mq + row, n = n0 + col;
                    const bool live = idx < total && m < p.M;
                    off[i] = live ? row_off(m) + n : -1;
                    v[i] = live ? sC[row * ldc + col] : 0.0f;
                    bias[i] = live && e.has_bias ? load_as_f32(e.bias_ptr, e.bias_dtype, n) : 0.0f;
                    tt[i] = live && tload ? load_as_f32(e.t_ptr, e.t_dtype, off[i]) : 0.0f;
                }
                finish<4>(e, v, bias, tt);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (off[i] >= 0) store_from_f32(p.y, p.y_dtype, off[i], v[i]);
            }
            return;
        }
        if (!e.simple) {
            // element by element along the fastest axis of the result
#pragma unroll 1
            for (int idx = t; idx < 32 * BN; idx += 256) {
                const int col = chan_fast ? idx % BN : idx / 32, row = chan_fast ? idx / BN : idx % 32;
                const int m = mq + row, n = n0 + col;
                if (m >= p.M || n >= p.N) continue;
                const int img = p.OHW == 1 ? m : (int)(__umulhi((uint32_t)m, p.div_ohw_mul) >> p.div_ohw_sh);
                const int64_t off = (int64_t)img * p.ys_n + (int64_t)(m - img * p.OHW) * p.ys_p + (int64_t)n * p.ys_c;
                float val = sC[row * ldc + col];
                for (int s = 0; s < e.n_ops; ++s) val = epi_step(e, s, val, off, n);
                store_from_f32(p.y, p.y_dtype, off, val);
            }
            return;
        }
        if (p.ys_p == 1 && (p.OHW & 3) == 0 && (p.ys_c & 3) == 0 && (p.ys_n & 3) == 0 && (((uintptr_t)p.y | (uintptr_t)e.t_ptr) & 15) == 0) {
            // four pixels (m a multiple of four: never across an image) of one channel per thread; 8 groups of pixels x 32 channels
            const int row = (t & 7) * 4, m = mq + row;
            if (m >= p.M) return;                         // M is a multiple of four here
            const int img = (int)(__umulhi((uint32_t)m, p.div_ohw_mul) >> p.div_ohw_sh);
            const int64_t base = (int64_t)img * p.ys_n + (m - img * p.OHW);
#pragma unroll 1
            for (int col = t >> 3; col < BN; col += 32) {
                const int n = n0 + col;
                if (n >= p.N) break;
                const int64_t off = base + (int64_t)n * p.ys_c;
                float v[4], bias[4], tt[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                if (tload && e.t_dtype == DT_F32) {
                    const f32x4 f = *(const f32x4 *)((const float *)e.t_ptr + off);
#pragma unroll
                    for (int k = 0; k < 4; ++k) tt[k] = f[k];
                } else if (tload) {
                    const u32x2 h = *(const u32x2 *)((const uint16_t *)e.t_ptr + off);
#pragma unroll
                    for (int k = 0; k < 4; ++k) tt[k] = __uint_as_float((k & 1) ? h[k >> 1] & 0xffff0000u : h[k >> 1] << 16);
                }
                const float b = e.has_bias ? load_as_f32(e.bias_ptr, e.bias_dtype, n) : 0.0f;
#pragma unroll
                for (int k = 0; k < 4; ++k) { bias[k] = b; v[k] = sC[(row + k) * ldc + col]; }
                finish<4>(e, v, bias, tt);
                if (p.y_dtype == DT_F32) *(f32x4 *)((float *)p.y + off) = f32x4{v[0], v[1], v[2], v[3]};
                else *(u32x2 *)((uint16_t *)p.y + off) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
            }
            return;
        }
        const int row = t & 31, m = mq + row;
        if (m >= p.M) return;
        const int img = p.OHW == 1 ? m : (int)(__umulhi((uint32_t)m, p.div_ohw_mul) >> p.div_ohw_sh);
        const int64_t base = (int64_t)img * p.ys_n + (int64_t)(m - img * p.OHW) * p.ys_p;
#pragma unroll 1
        for (int c0 = t >> 5; c0 < BN; c0 += 32) {
            if (n0 + c0 >= p.N) break;
            float v[4], bias[4], tt[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = n0 + c0 + 8 * i;
                tt[i] = bias[i] = 0.0f;
                v[i] = sC[row * ldc + c0 + 8 * i];
                if (n >= p.N) continue;
                if (e.has_bias) bias[i] = load_as_f32(e.bias_ptr, e.bias_dtype, n);
                if (tload) tt[i] = load_as_f32(e.t_ptr, e.t_dtype, base + (int64_t)n * p.ys_c);
            }
            finish<4>(e, v, bias, tt);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (n0 + c0 + 8 * i < p.N) store_from_f32(p.y, p.y_dtype, base + (int64_t)(n0 + c0 + 8 * i) * p.ys_c, v[i]);
        }
    }

    // LSTM gate math: packed column g*(BN/4)+u of the tile holds gate g of hidden unit bn*(BN/4)+u
    static __device__ __forceinline__ void gates_pass(const IgemmParams &p, const float *sC, int ldc, int t, int mq, int bn)
    {
        const Epilogue &e = p.epi;
        constexpr int U = BN / 4;
        for (int idx = t; idx < 32 * U; idx += 256) {
            int row = idx / U, u = idx - row * U;
            int m = mq + row, unit = bn * U + u;
            if (m < p.M && unit < p.hidden) {
                float z[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    z[g] = sC[row * ldc + g * U + u];
                    for (int s = 0; s < e.n_ops; ++s)      // only E_BIAS steps reach a gate epilogue
                        z[g] += load_as_f32(epi_ptr(e, epi_arg(e, s)), epi_ptr_dtype(e, epi_arg(e, s)), g * p.hidden + unit);
                }
                float c_old = p.c_in[(int64_t)m * p.hidden + unit];
                float cn = sigmoidf_(z[1]) * c_old + sigmoidf_(z[0]) * tanhf_(z[2]);
                float hn = sigmoidf_(z[3]) * tanhf_(cn);
                p.c_out[(int64_t)m * p.hidden + unit] = cn;
                store_from_f32(p.h_out, p.h_dtype, (int64_t)m * p.hidden + unit, hn);
            }
        }
    }
};

// Results in Shape order (pixels fastest) behind a simple chain: a thread's pixels and channels, fixed for the whole tile, so that
// what the chain reads of them can be requested long before they are finished.
//   PE_VEC    four pixels of one channel (whole groups of four per image): 8 groups of pixels x 32 channels per pass of 32 rows
//   PE_PIXEL  one pixel: 32 pixels x 8 channels
enum { PE_NONE = 0, PE_VEC, PE_PIXEL };
template <int BM, int BN>
struct PixelEpilogue {
    static constexpr int NQ = BM / 32, NV = BN / 32, NP = BN / 8;      // passes; channels per thread and pass of either form
    int form;
    uint32_t raw[NQ * NP];                 // PE_VEC: 4 words per (pass, channel) or 2 in bf16; PE_PIXEL: one
    float bias[NP];

    static __device__ __forceinline__ int64_t base(const IgemmParams &p, int m)
    {
        const int img = p.OHW == 1 ? m : (int)(__umulhi((uint32_t)m, p.div_ohw_mul) >> p.div_ohw_sh);
        return (int64_t)img * p.ys_n + (m - img * p.OHW);
    }

    __device__ __forceinline__ void request(const IgemmParams &p, int t, int m0, int n0)
    {
        const Epilogue &e = p.epi;
        form = PE_NONE;
        // a bias or a residual, and half a tile of channels at least (without either the rolled passes are up to 1.1x ahead, and on few channels)
        if (!e.simple || (e.t_op < 0 && !e.has_bias) || p.N - n0 < BN / 2 || p.ys_p != 1 || p.ys_c == 1 || p.splits > 1) return;
        const bool vec = (p.OHW & 3) == 0 && (p.ys_c & 3) == 0 && (p.ys_n & 3) == 0 && (((uintptr_t)p.y | (uintptr_t)e.t_ptr) & 15) == 0;
        form = vec ? PE_VEC : PE_PIXEL;
        const int row = vec ? (t & 7) * 4 : t & 31, c0 = vec ? t >> 3 : t >> 5, step = vec ? 32 : 8;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int n = n0 + c0 + step * j;
            bias[j] = e.has_bias && c0 + step * j < BN && n < p.N ? load_as_f32(e.bias_ptr, e.bias_dtype, n) : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < NQ * NP; ++i) raw[i] = 0u;
        if (e.t_op < 0) return;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int m = m0 + q * 32 + row;
            const int64_t b = base(p, m);
            if (vec) {
#pragma unroll
                for (int j = 0; j < NV; ++j) {
                    const int n = n0 + c0 + 32 * j;
                    if (m >= p.M || n >= p.N) continue;
                    const int64_t off = b + (int64_t)n * p.ys_c;
                    if (e.t_dtype == DT_F32) {
                        const u32x4 f = *(const u32x4 *)((const float *)e.t_ptr + off);
#pragma unroll
                        for (int k = 0; k < 4; ++k) raw[q * NP + 4 * j + k] = f[k];
                    } else {
                        const u32x2 h = *(const u32x2 *)((const uint16_t *)e.t_ptr + off);
                        raw[q * NP + 4 * j] = h[0];
                        raw[q * NP + 4 * j + 1] = h[1];
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    const int n = n0 + c0 + 8 * j;
                    if (m >= p.M || n >= p.N) continue;
                    const int64_t off = b + (int64_t)n * p.ys_c;
                    raw[q * NP + j] = e.t_dtype == DT_F32 ? ((const uint32_t *)e.t_ptr)[off] : (uint32_t)((const uint16_t *)e.t_ptr)[off];
                }
            }
        }
    }

    // the pass's 32 rows from sC, BN + 1 floats apart
    __device__ __forceinline__ void store(const IgemmParams &p, const float *sC, int t, int m0, int n0, int q)
    {
        const Epilogue &e = p.epi;
        const bool vec = form == PE_VEC, f32 = e.t_dtype == DT_F32;
        const int row = vec ? (t & 7) * 4 : t & 31, c0 = vec ? t >> 3 : t >> 5;
        const int m = m0 + q * 32 + row;
        if (m >= p.M) return;
        const int64_t b = base(p, m);
        if (vec) {
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const int c = c0 + 32 * j, n = n0 + c;
                if (n >= p.N) continue;
                float v[4], bs[4], tt[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    v[k] = sC[(row + k) * (BN + 1) + c];
                    bs[k] = bias[j];
                    const uint32_t w = raw[q * NP + 4 * j + (k >> 1)];
                    tt[k] = f32 ? __uint_as_float(raw[q * NP + 4 * j + k]) : __uint_as_float(k & 1 ? w & 0xffff0000u : w << 16);
                }
                TileEpilogue<64>::template finish<4>(e, v, bs, tt);
                const int64_t off = b + (int64_t)n * p.ys_c;
                if (p.y_dtype == DT_F32) *(f32x4 *)((float *)p.y + off) = f32x4{v[0], v[1], v[2], v[3]};
                else *(u32x2 *)((uint16_t *)p.y + off) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
            }
            return;
        }
        float v[NP], tt[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            v[j] = sC[row * (BN + 1) + c0 + 8 * j];
            tt[j] = __uint_as_float(f32 ? raw[q * NP + j] : raw[q * NP + j] << 16);
        }
        TileEpilogue<64>::template finish<NP>(e, v, bias, tt);
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int n = n0 + c0 + 8 * j;
            if (n < p.N) store_from_f32(p.y, p.y_dtype, b + (int64_t)n * p.ys_c, v[j]);
        }
    }
};

}  // namespace rl
