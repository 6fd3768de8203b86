// Both gradients of a layer in one launch: the contraction that gives the gradient of its input (igemm_dma.h) and the one over the
// rows of both operands that gives the gradient of its weights (igemm_tn.h), 64x64 tiles of either, three workgroups per CU.
//
// Neither needs the other's result, and each alone ends in a last round that leaves CUs idle, then in the 3 to 4 us that pass between
// dependent launches.  Together the workgroups of the one fill the rounds of the other.  The ones with the longer K loop come
// first in the grid.  Dense 512 x 1000 x 784 bf16 15.1 -> 10.2 us; 32x64x28x28 -> 64 3x3 f32 60 -> 50, with the slices cut for the
// shared launch (Planner::reslice_beside); of 900 drawn backward passes 355 go this way, at 0.81 (dense bf16), 0.84 (dense f32), 0.75 (conv
// bf16) and 0.85 (conv f32) of the time without shared launches (no_pair; a convolution's layout changes share one too).
#include <algorithm>

#include "igemm_dma.h"
#include "igemm_tn.h"

namespace rl {

// The contraction over rows, in the grid of the other one.  Its workgroups or the other's are the first n_first.
template <bool CONV> struct BesideRows {
    static constexpr bool other = true;
    TnParams q;
    int32_t n_first, rows_first;

    template <typename T, int STAGE>
    __device__ __forceinline__ bool take(int &bid, unsigned char (&st0)[STAGE], unsigned char (&st1)[STAGE], unsigned char (&st2)[STAGE]) const
    {
        static_assert(STAGE == tn_stage_bytes<64, 64>(), "one set of stages for either");
        // the second part starts at a multiple of the XCD count, so that a workgroup's XCD is that of its number in its own part
        const int start = (n_first + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
        const bool first = bid < start;
        if (!first) bid -= start;
        if (first != (rows_first != 0)) return true;
        if (bid < q.nblk_m * q.nblk_n * q.splits) igemm_tn_body<T, 64, 64, CONV>(q, bid, st0, st1, st2);
        return false;
    }
};

#define RL_ONE(T, MODE, TAPS, CONV) template __global__ void igemm_dma_kernel<T, 64, 64, MODE, TAPS, BesideRows<CONV>, 1>(const IgemmParams, const BesideRows<CONV>);
#define RL_INST(T, MODE) RL_ONE(T, MODE, false, false) RL_ONE(T, MODE, false, true) RL_ONE(T, MODE, true, true)
RL_INST(float, STORE_ROWS) RL_INST(float, STORE_ANY) RL_INST(uint16_t, STORE_ROWS) RL_INST(uint16_t, STORE_ANY)
#undef RL_INST
#undef RL_ONE

bool igemm_dma_takes(const IgemmParams &p, bool taps, int element_size);        // igemm_dma.hip
bool igemm_dma_splits_ok(const IgemmParams &p, bool taps, int element_size);
bool igemm_tn_prepare(TnParams &p, int element_size, int tile);                 // igemm_tn.hip
hipError_t launch_tn_reduce(const TnParams &p, hipStream_t s);
hipError_t launch_splitk_reduce(const IgemmParams &p, hipStream_t s);           // igemm_dma.hip

template <typename T>
static hipError_t launch_typed(const IgemmParams &p, const TnParams &q, bool taps, hipStream_t s)
{
    const bool rows = p.splits > 1 || (p.ys_n == (int64_t)p.OHW * p.ys_p && p.ys_c == 1 && (p.N & 7) == 0 && (p.ys_p & 7) == 0);
    const int nk = (p.K + 128 / (int)sizeof(T) - 1) / (128 / (int)sizeof(T));
    const int64_t na = (int64_t)p.nblk_m * p.nblk_n * std::max(p.splits, 1), nb = (int64_t)q.nblk_m * q.nblk_n * q.splits;
    const int rows_first = q.split_tiles > (p.splits > 1 ? p.split_tiles : nk);
    const int64_t first = rows_first ? nb : na, grid = (first + NUM_XCD - 1) / NUM_XCD * NUM_XCD + (rows_first ? na : nb);
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
#define RL_GO(MODE, TAPS, CONV) hipLaunchKernelGGL((igemm_dma_kernel<T, 64, 64, MODE, TAPS, BesideRows<CONV>, 1>), dim3((unsigned)grid), dim3(256), 0, s, p, (BesideRows<CONV>{q, (int)first, rows_first}))
    if (taps && rows) RL_GO(STORE_ROWS, true, true);
    else if (taps) RL_GO(STORE_ANY, true, true);
    else if (q.conv && rows) RL_GO(STORE_ROWS, false, true);
    else if (q.conv) RL_GO(STORE_ANY, false, true);
    else if (rows) RL_GO(STORE_ROWS, false, false);
    else RL_GO(STORE_ANY, false, false);
#undef RL_GO
    return hipGetLastError();
}

bool igemm_grads_ok(const IgemmParams &a, const IgemmLaunch &la, const TnParams &b, int32_t tn_dtype, int32_t tn_tile)
{
    return la.dma && la.tile == TILE_64x64 && !la.lp && !la.gates && !la.direct && a.in_dtype == tn_dtype && tn_tile == 64 && (!la.taps || b.conv);
}

hipError_t launch_igemm_grads(const IgemmParams &a, const IgemmLaunch &la, const TnParams &b, int32_t dtype, hipStream_t s)
{
    IgemmParams p = a;
    TnParams q = b;
    const int es = dtype == DT_BF16 ? 2 : 4;
    if (!igemm_grads_ok(a, la, b, dtype, 64) || !igemm_dma_takes(p, la.taps, es) || !igemm_tn_prepare(q, es, 64)) return hipErrorInvalidValue;
    p.nblk_m = (p.M + 63) / 64;
    p.nblk_n = (p.N + 63) / 64;
    if ((int64_t)p.nblk_m * p.nblk_n > 0x7fffffff) return hipErrorInvalidValue;
    if (p.splits > 1 && !igemm_dma_splits_ok(p, la.taps, es)) return hipErrorInvalidValue;
    hipError_t er = dtype == DT_BF16 ? launch_typed<uint16_t>(p, q, la.taps, s) : launch_typed<float>(p, q, la.taps, s);
    if (er == hipSuccess && p.splits > 1) er = launch_splitk_reduce(p, s);
    if (er != hipSuccess || q.splits == 1) return er;
    return launch_tn_reduce(q, s);
}

}  // namespace rl
