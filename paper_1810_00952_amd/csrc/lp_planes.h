// How a wave of the pixel-on-lane kernels stores its tile in Shape order (pixels fastest): accumulators plus bias parked in LDS a
// channel's pixels in a row, read back four pixels at a time, ReLU, one rounding, 8-byte stores: 64 or 128 contiguous bytes a channel.
// In place of whole rows of channels and a transposition behind them, which reads and writes the result once more and is a
// launch of its own.  Images of whole groups of four pixels; a residual comes in the same order, requested ahead of the K loop.
// bf16, before and after: 64x128x28x28 -> 128 3x3 33.5 -> 26.3 us, 32x64x56x56 -> 192 1x1 46.9 -> 28.9, 16x64x28x28 -> 128 14.3 -> 10.4;
// 14 layers of the range to 0.62 .. 0.88 of their time, none slower.  With a channel-first
// residual, which then is not turned either: 43.6 -> 27.8, 70.0 -> 40.2, 17.5 -> 10.7; 13 layers to 0.53 .. 0.80.
#pragma once
#include "device_utils.h"

namespace rl {

// m0, n0: the wave's first pixel and channel
template <int WTM, int WTN> struct PlanesTile {
    static constexpr uint32_t OUT = 0x80000000u;
    static constexpr int LPC = WTM / 4, CPP = 64 / LPC, NQ = WTN / CPP;      // lanes per channel, channels per pass, passes
    uint32_t off, step;                               // of the lane's pixels and first channel; from pass to pass
    u32x2 res[NQ];

    // NQ loads; without a residual from an empty descriptor: zeros, no memory traffic
    __device__ __forceinline__ void request(const IgemmParams &p, int m0, int n0, int lane, __amdgpu_buffer_rsrc_t rres)
    {
#if defined(__HIP_DEVICE_COMPILE__)
        const int ch = lane / LPC, m = m0 + 4 * (lane % LPC);
        const int img = p.OHW == 1 ? m : (int)(__umulhi((uint32_t)m, p.div_ohw_mul) >> p.div_ohw_sh);
        off = m < p.M ? (uint32_t)(((int64_t)img * p.ys_n + (m - img * p.OHW) + (int64_t)(n0 + ch) * p.ys_c) * 2) : OUT;
        step = (uint32_t)(CPP * p.ys_c * 2);
#pragma unroll
        for (int q = 0; q < NQ; ++q) res[q] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rres, n0 + ch + CPP * q < p.N ? off + (uint32_t)q * step : OUT, 0, 0));
#endif
    }

    // park: the wave's WTM * WTN * 4 bytes of LDS; ry: the result's descriptor
    __device__ __forceinline__ void store(const IgemmParams &p, unsigned char *park, const f32x16 (&acc)[WTM / 32][WTN / 32], const f32x4 (&bias)[WTN / 32][4], int n0, int lane,
                                          __amdgpu_buffer_rsrc_t ry, float lo)
    {
#if defined(__HIP_DEVICE_COMPILE__)
        float *pk = (float *)park;
        const int epix = lane & 31, ehalf = lane >> 5, px = 4 * (lane % LPC), ch = lane / LPC;
#pragma unroll
        for (int i = 0; i < WTM / 32; ++i)
#pragma unroll
            for (int j = 0; j < WTN / 32; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    pk[(j * 32 + 8 * (r >> 2) + 4 * ehalf + (r & 3)) * WTM + i * 32 + epix] = acc[i][j][r] + bias[j][r >> 2][r & 3];
        wave_lds_exchange();
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            f32x4 v = *(const f32x4 *)(pk + (ch + CPP * q) * WTM + px);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] += __uint_as_float(k & 1 ? res[q][k >> 1] & 0xffff0000u : res[q][k >> 1] << 16);
            const u32x2 o = {pack_bf16x2(fmaxf(v[0], lo), fmaxf(v[1], lo)), pack_bf16x2(fmaxf(v[2], lo), fmaxf(v[3], lo))};
            __builtin_amdgcn_raw_buffer_store_b64(o, ry, n0 + ch + CPP * q < p.N ? off + (uint32_t)q * step : OUT, 0, 0);
        }
#endif
    }
};

}  // namespace rl
