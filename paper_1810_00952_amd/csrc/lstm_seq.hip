// A whole LSTM sequence in one launch, input projections already done (zx of every step, packed column order):
//
//   z_t = zx_t + h_{t-1} . Wh^T + bias;  c_t, h_t by the gates (see lstm_step.hip)
//
// What bounds the one-launch-per-step form is not its arithmetic: 6.3 us per step, of which about 3 pass between dependent
// launches and the rest fetching 128 KB per CU again (64 KB of weights that never change).  Here every CU keeps its weights in
// registers for the whole sequence and a step costs one exchange of h between the CUs that need it: about 2.7 us at 64 rows of
// 1024 units (128 steps with their projections: 825 us step by step, 417 us here; 383 us if the 134 MB of projections still
// stand in the last-level cache).  What is left of a step is a chain of latencies - the flags' poll, the L2 round trip for h,
// the meeting of the partial sums, the gates, the store's acknowledgement - and not work: the MFMAs of a step take 0.3 us.
//
// Split: batch rows over the eight XCDs (8 of 64), hidden units over the CUs of an XCD (32 each at H = 1024).  Inside a CU each
// of the four waves multiplies all 128 gate columns by its quarter of H (256 registers of weights per lane at H = 1024), so that
// h is fetched once per CU, each wave its own part straight into registers; the four partial sums meet in LDS.  (Eight units
// per wave over the whole of H, with h staged in LDS: 520 us.  Quarters with the loads left to the compiler, which asks for h two
// fragments at a time and for the projections only after the products: 548 us.)
// A step's h is written and read inside one XCD, through its L2: the stores go there (the vector L1 writes through), the loads
// bypass the L1 (device scope; the narrower scopes may hit it).  No cache is flushed, which is what made a grid-wide barrier
// cost more than a launch.  A workgroup publishes step t by writing t + 1 into its flag word after its stores were acknowledged;
// the members of its group poll the flags of all of them.
// MFMA 16x16x32, weights as the row operand with row 4u + gate: a lane's four result registers are the four gates of one
// (unit, batch row), so the gates, c (in registers throughout) and h need no exchange between lanes.
//
// Waiting for other workgroups is safe only if all of them are resident.  The kernel is launched cooperatively, and it checks:
// every workgroup registers (device-scope atomics); the last one finds `members` workgroups on every XCD and says "go", or says
// "alone"; so does anyone whose bounded wait for the others runs out.  Alone, a workgroup takes sixteen batch rows through the
// whole sequence by itself (weights fetched every step: slow, but it waits for nobody).
// The control words live where step T-1's projections of batch row 0 begin (scratch); what they displace was saved at the start
// of h_{T-1} (of h_{T-2} where h0 lies there) by the launch before and is fetched into LDS before registering.
#include "device_utils.h"

namespace rl {

namespace {

typedef __amdgpu_buffer_rsrc_t rsrc_t;
#define RL_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

__device__ __forceinline__ rsrc_t make_rsrc(const void *ptr, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)ptr, 0, bytes, 0x00020000);   // raw buffer, untyped dwords
}

__device__ __forceinline__ void wg_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

constexpr int N_XCD = 8, DEV = 16;              // DEV: cache policy (sc1, device scope) of a load that bypasses the vector L1
constexpr int CTL_TOTAL = N_XCD, CTL_STATE = N_XCD + 1, CTL_FLAGS = 32;
enum { ST_WAIT = 0, ST_GO = 1, ST_ALONE = 2 };
constexpr int UNITS = 32;                       // hidden units of a workgroup
constexpr int MAX_POLLS = 1 << 20;              // of a resident workgroup for its group: never reached; ends the wait, with NaN in c, all the same

}  // namespace

int lstm_seq_ctl_words(int H) { return CTL_FLAGS + N_XCD * (H / UNITS); }

// saves the words the control block displaces and clears it, or puts them back
__global__ void lstm_seq_prepare_kernel(uint32_t *ctl, uint32_t *save, int words, int back)
{
    for (int i = threadIdx.x; i < words; i += blockDim.x) {
        if (back) ctl[i] = save[i];
        else { save[i] = ctl[i]; ctl[i] = 0u; }
    }
}

// KS: H / 32.  HALF: at most eight rows per XCD, so that half of the MFMA's sixteen columns are empty: the lanes of those take
// every other unit in the gate arithmetic, which is a serial chain of exponentials (128 steps of 64 rows, projections in cache: 498 -> 446 us).
template <int KS, bool HALF>
__global__ __launch_bounds__(256, 1) void lstm_seq_kernel(const LstmSeqParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub; the body uses gfx950-only builtins
    constexpr int H = KS * 32, MEMBERS = H / UNITS, ROWB = H * 2;
    __shared__ __attribute__((aligned(1024))) unsigned char hbuf[2][16 * ROWB];
    __shared__ f32x4 part[4][UNITS / 4][64];    // the waves' partial sums
    __shared__ uint32_t saved[CTL_FLAGS + N_XCD * MEMBERS];
    __shared__ int s_state, s_slot;

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int l16 = lane & 15, q4 = lane >> 4;
    uint32_t *ctl = p.ctl;
    const int words = CTL_FLAGS + N_XCD * MEMBERS;
    for (int i = t; i < words; i += 256) saved[i] = p.save[i];
    uint32_t xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    xcc &= N_XCD - 1;
    __syncthreads();                             // the saved words are fetched before anyone can pass the registration

    if (t == 0) {
        s_slot = (int)__hip_atomic_fetch_add(ctl + xcc, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t before = __hip_atomic_fetch_add(ctl + CTL_TOTAL, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (before == gridDim.x - 1) {
            bool even = true;
            for (int i = 0; i < N_XCD; ++i) even &= __hip_atomic_load(ctl + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)MEMBERS;
            uint32_t want = ST_WAIT;
            __hip_atomic_compare_exchange_strong(ctl + CTL_STATE, &want, even ? ST_GO : ST_ALONE, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        uint32_t st = ST_WAIT;
        for (int i = 0; i < p.spins && st == ST_WAIT; ++i) st = __hip_atomic_load(ctl + CTL_STATE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (st == ST_WAIT) {
            uint32_t want = ST_WAIT;
            if (__hip_atomic_compare_exchange_strong(ctl + CTL_STATE, &want, (uint32_t)ST_ALONE, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) st = ST_ALONE;
            else st = want;
        }
        s_state = (int)st;
    }
    __syncthreads();
    const bool go = __builtin_amdgcn_readfirstlane(s_state) == ST_GO;
    const int member = __builtin_amdgcn_readfirstlane(s_slot);

    // ---- rows and units of this workgroup
    const int R = go ? (p.B + N_XCD - 1) / N_XCD : 16;           // at most 16 (checked by the launcher)
    const int r0 = (go ? (int)xcc : (int)blockIdx.x) * R;
    const int rows = min(R, p.B - r0);
    if (rows <= 0 || (go && member >= MEMBERS)) return;
    const bool live = l16 < rows;
    int row = r0 + min(l16, rows - 1);                           // the lane's batch row
    const int N = 4 * H;
    const rsrc_t rw = make_rsrc(p.w, p.w_bytes);
    // packed weight row (= packed column of zx) of (unit, gate)
    auto packed = [](int unit, int gate) { return (unit >> 4) * 64 + gate * 16 + (unit & 15); };
    auto zx_at = [&](int tt, int unit, int gate) -> float {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(make_rsrc(p.zx + (size_t)tt * p.B * N, (uint32_t)p.B * N * 4u), (uint32_t)(row * N + packed(unit, gate)) * 4u, 0, 0));
    };
    auto zx_true = [&](float z, int tt, int unit, int gate) -> float {       // ... unless the control words stand there
        const int col = packed(unit, gate);
        return tt == p.T - 1 && row == 0 && col < words ? __uint_as_float(saved[col]) : z;
    };
    // h_{tt-1} of the workgroup's rows into buffer tt & 1; 16-byte chunk c of row r at position c ^ 4 (r & 3)
    auto fetch_h = [&](int tt) {
        const char *src = tt == 0 ? (const char *)p.h0 : (const char *)p.h_seq + (size_t)(tt - 1) * p.h_step_bytes;
        const rsrc_t rh = make_rsrc(src + (size_t)r0 * ROWB, (uint32_t)rows * ROWB);
        constexpr int PER = (ROWB + 1023) / 1024;                // direct loads per row, 1 KB each (the last may be half used)
        for (int i = wave; i < rows * PER; i += 4) {
            const int r = i / PER, part = i - r * PER, at = part * 64 + lane;
            if (at < ROWB / 16)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rh, RL_LDS_PTR(hbuf[tt & 1] + r * ROWB + part * 1024), 16, (uint32_t)(r * ROWB + (at ^ ((r & 3) << 2)) * 16), 0, 0, DEV);
        }
        asm volatile("" ::: "memory");                           // what is requested next stays behind these in the counter
    };
    const int hrow = min(l16, rows - 1);
    const int h_key = (hrow & 3) << 2;
    auto h_frag = [&](int tt, int ks) -> bf16x8 {
        return __builtin_bit_cast(bf16x8, *(const u32x4 *)(hbuf[tt & 1] + hrow * ROWB + (((ks * 4 + q4) ^ h_key) << 4)));
    };
    auto bias_at = [&](int unit, int gate) { return p.bias ? p.bias[gate * H + unit] : 0.0f; };

    if (go) {
        // A wave multiplies all 128 gate columns by its quarter of H (its h fragments come straight from the L2 into registers), the
        // quarters meet in LDS, and it finishes eight of the units.
        constexpr int KW = KS / 4, CT = UNITS / 4;
        const int unit0 = member * UNITS + wave * 8;
        u32x4 fw[CT][KW];                                         // row l16 = 4 unit + gate of column tile ct, contraction indices 32 (wave KW + ks) + 8 q4 ..
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const uint32_t wrow = (uint32_t)packed(member * UNITS + ct * 4 + (l16 >> 2), l16 & 3) * (uint32_t)p.Kp * 2u + (uint32_t)p.k_off * 2u + (uint32_t)(wave * KW * 64 + q4 * 16);
#pragma unroll
            for (int ks = 0; ks < KW; ++ks) fw[ct][ks] = __builtin_amdgcn_raw_buffer_load_b128(rw, wrow + ks * 64, 0, 0);
        }
        const uint32_t h_off = live ? (uint32_t)(l16 * ROWB + wave * KW * 64 + q4 * 16) : 0x80000000u;     // lanes past the rows read zeros
        // what the lane finishes: unit tile 2 wave + ct_of(u) of its batch row
        constexpr int NU = HALF ? 1 : 2;
        const int grow = HALF ? l16 & 7 : l16;                    // row of the group, and the lane that holds its sums
        const int src_lane = q4 * 16 + grow;
        const bool glive = grow < rows;
        row = r0 + min(grow, rows - 1);
        auto ct_of = [&](int u) { return HALF ? l16 >> 3 : u; };
        float bias_r[NU][4], c_r[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int unit = unit0 + ct_of(u) * 4 + q4;
#pragma unroll
            for (int g = 0; g < 4; ++g) bias_r[u][g] = bias_at(unit, g);
            c_r[u] = p.c[(size_t)row * H + unit];
        }
        float z_r[2][NU][4];                                      // projections of step t and t + 1 (set t & 1)
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int g = 0; g < 4; ++g) z_r[0][u][g] = zx_at(0, unit0 + ct_of(u) * 4 + q4, g);
        uint32_t *flags = ctl + CTL_FLAGS + xcc * MEMBERS;
        const rsrc_t rf = make_rsrc(flags, MEMBERS * 4);
        bool lost = false;
        auto step = [&](int tt, float (&zc)[NU][4], float (&zn)[NU][4]) {
            if (tt > 0) {
                // every member's flag says its h_{tt-1} is in the L2 (lanes past the members read zero and do not count)
                int i = 0;
#pragma unroll 1
                for (; i < MAX_POLLS; ++i) {
                    const uint32_t f = __builtin_amdgcn_raw_buffer_load_b32(rf, (uint32_t)lane * 4u, 0, DEV);
                    if (__all(lane >= MEMBERS || f >= (uint32_t)tt)) break;
                    asm volatile("" ::: "memory");
                }
                lost |= i == MAX_POLLS;
            }
            const char *src = tt == 0 ? (const char *)p.h0 : (const char *)p.h_seq + (size_t)(tt - 1) * p.h_step_bytes;
            const rsrc_t rh = make_rsrc(src + (size_t)r0 * ROWB, (uint32_t)rows * ROWB);
            u32x4 hf[KW];
#pragma unroll
            for (int ks = 0; ks < KW; ++ks) hf[ks] = __builtin_amdgcn_raw_buffer_load_b128(rh, h_off + ks * 64, 0, DEV);
            __builtin_amdgcn_sched_barrier(0);                   // all of them in flight at once; left to itself the compiler asks for two at a time
            const int tn = min(tt + 1, p.T - 1);
#pragma unroll
            for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int g = 0; g < 4; ++g) zn[u][g] = zx_at(tn, unit0 + ct_of(u) * 4 + q4, g);
            __builtin_amdgcn_sched_barrier(0);                   // the next step's projections are requested here, behind h, and not after the products
            f32x4 acc[CT];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) acc[ct] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < KW; ++ks)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
                    acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fw[ct][ks]), __builtin_bit_cast(bf16x8, hf[ks]), acc[ct], 0, 0, 0);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) part[wave][ct][lane] = acc[ct];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            wg_barrier();
            f32x4 z[NU];
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int at = wave * 2 + ct_of(u);
                z[u] = (part[0][at][src_lane] + part[1][at][src_lane]) + (part[2][at][src_lane] + part[3][at][src_lane]);
            }
            if (tt == p.T - 1 && r0 == 0) {
#pragma unroll
                for (int u = 0; u < NU; ++u)
#pragma unroll
                    for (int g = 0; g < 4; ++g) zc[u][g] = zx_true(zc[u][g], tt, unit0 + ct_of(u) * 4 + q4, g);
            }
            uint16_t *out = (uint16_t *)((char *)p.h_seq + (size_t)tt * p.h_step_bytes) + (size_t)row * H;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
#pragma unroll
                for (int g = 0; g < 4; ++g) z[u][g] = (z[u][g] + zc[u][g]) + bias_r[u][g];
                c_r[u] = sigmoidf_(z[u][1]) * c_r[u] + sigmoidf_(z[u][0]) * tanhf_(z[u][2]);
                const float hn = sigmoidf_(z[u][3]) * tanhf_(c_r[u]);
                if (glive) out[unit0 + ct_of(u) * 4 + q4] = (uint16_t)f32_to_bf16_bits(hn);
            }
            // this wave's h is in the L2; after the barrier every wave's is (and every wave has read the partial sums)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            wg_barrier();
            if (t == 0) __hip_atomic_store(flags + member, (uint32_t)(tt + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
#pragma unroll 1
        for (int tt = 0; tt < p.T; tt += 2) {
            step(tt, z_r[0], z_r[1]);
            if (tt + 1 < p.T) step(tt + 1, z_r[1], z_r[0]);
            if (lost) break;
        }
#pragma unroll
        for (int u = 0; u < NU; ++u)
            if (glive) p.c[(size_t)row * H + unit0 + ct_of(u) * 4 + q4] = lost ? __uint_as_float(0x7fc00000u) : c_r[u];
        return;
    }

    // ---- alone: sixteen rows, every unit; the wave's units are 4 wave, 4 wave + 16, ...
#pragma unroll 1
    for (int tt = 0; tt < p.T; ++tt) {
        if (tt == 0) {
            fetch_h(0);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        __syncthreads();
        uint16_t *out = (uint16_t *)((char *)p.h_seq + (size_t)tt * p.h_step_bytes) + (size_t)row * H;
#pragma unroll 1
        for (int u0 = wave * 4; u0 < H; u0 += 16) {
            f32x4 acc[2] = {f32x4{0.0f, 0.0f, 0.0f, 0.0f}, f32x4{0.0f, 0.0f, 0.0f, 0.0f}};
            const uint32_t wrow = (uint32_t)packed(u0 + (l16 >> 2), l16 & 3) * (uint32_t)p.Kp * 2u + (uint32_t)p.k_off * 2u + (uint32_t)q4 * 16u;
#pragma unroll 8
            for (int ks = 0; ks < KS; ++ks)
                acc[ks & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rw, wrow + ks * 64, 0, 0)), h_frag(tt, ks), acc[ks & 1], 0, 0, 0);
            const int unit = u0 + q4;
            float z[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) z[g] = ((acc[0][g] + acc[1][g]) + zx_true(zx_at(tt, unit, g), tt, unit, g)) + bias_at(unit, g);
            if (live) {
                float *cp = p.c + (size_t)row * H + unit;
                const float cn = sigmoidf_(z[1]) * *cp + sigmoidf_(z[0]) * tanhf_(z[2]);
                const uint16_t hb = (uint16_t)f32_to_bf16_bits(sigmoidf_(z[3]) * tanhf_(cn));
                *cp = cn;
                out[unit] = hb;
                *(uint16_t *)(hbuf[(tt + 1) & 1] + l16 * ROWB + (((unit >> 3) ^ ((l16 & 3) << 2)) << 4) + (unit & 7) * 2) = hb;
            }
        }
    }
#endif
}

#define RL_INST(KS) template __global__ void lstm_seq_kernel<KS, false>(const LstmSeqParams); template __global__ void lstm_seq_kernel<KS, true>(const LstmSeqParams);
RL_INST(8) RL_INST(16) RL_INST(24) RL_INST(32)
#undef RL_INST

bool lstm_seq_ok(int64_t B, int64_t H, int64_t T) { return B >= 1 && B <= 16 * N_XCD && H >= 256 && H <= 1024 && H % 256 == 0 && T >= 8; }

hipError_t launch_lstm_seq(const LstmSeqParams &p0, hipStream_t s)
{
    LstmSeqParams p = p0;
    if (!lstm_seq_ok(p.B, p.H, p.T) || !p.h0 || !p.h_seq || !p.w || !p.zx || !p.c || !p.ctl || !p.save || p.spins < 0 || p.Kp < p.k_off + p.H || p.k_off < 0 || p.k_off % 8 != 0 ||
        p.Kp % 8 != 0 || (uint64_t)4 * p.H * p.Kp * 2 != p.w_bytes || p.w_bytes >= 0x7fffffffu || p.h_step_bytes < (size_t)p.B * p.H * 2 ||
        ((uintptr_t)p.ctl & 255) || ((uintptr_t)p.save & 3))
        return hipErrorInvalidValue;
    static const void *const kerns[4][2] = {{(const void *)lstm_seq_kernel<8, false>, (const void *)lstm_seq_kernel<8, true>}, {(const void *)lstm_seq_kernel<16, false>, (const void *)lstm_seq_kernel<16, true>},
                                            {(const void *)lstm_seq_kernel<24, false>, (const void *)lstm_seq_kernel<24, true>}, {(const void *)lstm_seq_kernel<32, false>, (const void *)lstm_seq_kernel<32, true>}};
    const void *kern = kerns[p.H / 256 - 1][p.B <= 8 * N_XCD];
    hipLaunchKernelGGL(lstm_seq_prepare_kernel, dim3(1), dim3(256), 0, s, p.ctl, p.save, lstm_seq_ctl_words(p.H), 0);
    hipError_t er = hipGetLastError();
    if (er != hipSuccess) return er;
    void *args[] = {&p};
    er = hipLaunchCooperativeKernel(kern, dim3((unsigned)(N_XCD * (p.H / UNITS))), dim3(256), args, 0, s);
    if (er == hipSuccess) return er;
    // this device cannot hold the grid (or has no cooperative launches): the projections as they were, for the caller's other form
    (void)hipGetLastError();
    hipLaunchKernelGGL(lstm_seq_prepare_kernel, dim3(1), dim3(256), 0, s, p.ctl, p.save, lstm_seq_ctl_words(p.H), 1);
    (void)hipGetLastError();
    return hipErrorNotSupported;
}

}  // namespace rl
