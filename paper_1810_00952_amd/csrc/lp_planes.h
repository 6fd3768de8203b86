// How a wave of the pixel-on-lane kernels stores its tile in Shape order (pixels fastest): accumulators plus bias parked in LDS a
// channel's pixels in a row, read back four pixels at a time, ReLU, one rounding, 8-byte stores: 64 or 128 contiguous bytes a channel.
// In place of whole rows of channels and a transposition behind them, which reads and writes the result once more and is a
// launch of its own.  Images of whole groups of four pixels; no residual (it would have to come in the same order).
// bf16, before and after: 64x128x28x28 -> 128 3x3 33.5 -> 26.3 us, 32x64x56x56 -> 192 1x1 46.9 -> 28.9, 16x64x28x28 -> 128 14.3 -> 10.4;
// 14 layers of the range to 0.62 .. 0.88 of their time, none slower.
#pragma once
#include "device_utils.h"

namespace rl {

// m0, n0: the wave's first pixel and channel; park: its WTM * WTN * 4 bytes of LDS; ry: the result's descriptor
template <int WTM, int WTN>
__device__ __forceinline__ void store_planes(const IgemmParams &p, unsigned char *park, const f32x16 (&acc)[WTM / 32][WTN / 32], const f32x4 (&bias)[WTN / 32][4], int m0, int n0,
                                             int lane, __amdgpu_buffer_rsrc_t ry, float lo)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr uint32_t OUT = 0x80000000u;
    constexpr int LPC = WTM / 4, CPP = 64 / LPC;      // lanes per channel, channels per pass
    float *pk = (float *)park;
    const int epix = lane & 31, ehalf = lane >> 5;
#pragma unroll
    for (int i = 0; i < WTM / 32; ++i)
#pragma unroll
        for (int j = 0; j < WTN / 32; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                pk[(j * 32 + 8 * (r >> 2) + 4 * ehalf + (r & 3)) * WTM + i * 32 + epix] = acc[i][j][r] + bias[j][r >> 2][r & 3];
    wave_lds_exchange();
    const int px = 4 * (lane % LPC), ch = lane / LPC, m = m0 + px;
    const int img = p.OHW == 1 ? m : (int)(__umulhi((uint32_t)m, p.div_ohw_mul) >> p.div_ohw_sh);
    const uint32_t off = m < p.M ? (uint32_t)(((int64_t)img * p.ys_n + (m - img * p.OHW) + (int64_t)(n0 + ch) * p.ys_c) * 2) : OUT;
    const uint32_t step = (uint32_t)(CPP * p.ys_c * 2);
#pragma unroll
    for (int q = 0; q < WTN / CPP; ++q) {
        const f32x4 v = *(const f32x4 *)(pk + (ch + CPP * q) * WTM + px);
        const u32x2 o = {pack_bf16x2(fmaxf(v[0], lo), fmaxf(v[1], lo)), pack_bf16x2(fmaxf(v[2], lo), fmaxf(v[3], lo))};
        __builtin_amdgcn_raw_buffer_store_b64(o, ry, n0 + ch + CPP * q < p.N ? off + (uint32_t)q * step : OUT, 0, 0);
    }
#endif
}

}  // namespace rl
