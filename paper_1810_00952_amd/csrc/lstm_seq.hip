// A whole LSTM sequence in one launch, input projections already done (zx of every step, packed column order):
//
//   z_t = zx_t + h_{t-1} . Wh^T + bias;  c_t, h_t by the gates (see lstm_step.hip)
//
// What bounds the one-launch-per-step form is not its arithmetic: 6.3 us per step, of which about 3 pass between dependent
// launches and the rest fetching 128 KB per CU again (64 KB of weights that never change).  Here every CU keeps its weights in
// registers for the whole sequence and a step costs one exchange of h between the CUs that need it: about 2.3 us at 64 rows of
// 1024 units (128 steps with their projections: 814 us step by step, 412 us here; 387 us if the 134 MB of projections still
// stand in the last-level cache).  What is left of a step is a chain of latencies - the flags' poll, the L2 round trip for h,
// the meeting of the partial sums, the gates, the store's acknowledgement - and not work: the MFMAs of a step take 0.3 us.
//
// Split: batch rows over the eight XCDs (8 of 64), hidden units over the CUs of an XCD (32 each at H = 1024).  Inside a CU each
// of the four waves multiplies all 128 gate columns by its quarter of H (256 registers of weights per lane at H = 1024), so that
// h is fetched once per CU, each wave its own part straight into registers; the four partial sums meet in LDS.  Wave w's quarter
// are the slices w, w + 4, ... of 64 contraction indices, summed and added up in the order of lstm_step.hip: the two forms give
// the same bits, so that which of them runs a sequence is a matter of time alone.  (Eight units
// per wave over the whole of H, with h staged in LDS: 520 us.  Quarters with the loads left to the compiler, which asks for h two
// fragments at a time and for the projections only after the products: 548 us.)
// A step's h is written and read inside one XCD, through its L2: the stores go there (the vector L1 writes through), the loads
// bypass the L1 (device scope; the narrower scopes may hit it).  No cache is flushed, which is what made a grid-wide barrier
// cost more than a launch.  A workgroup publishes step t by writing t + 1 into its flag word after its stores were acknowledged;
// the members of its group poll the flags of all of them.
// MFMA 16x16x32, weights as the row operand with row 4u + gate: a lane's four result registers are the four gates of one
// (unit, batch row), so the gates, c (in registers throughout) and h need no exchange between lanes.
//
// Waiting for other workgroups is safe only if they are resident.  So a workgroup first enters itself in the control block, and
// the first one to see all of them there closes the entry, or the first one that has waited longer than the sequence would take
// the workgroups that are there (3 us a step at full strength): they wait for no one else, whoever starts later returns at once.
// The XCDs that have workgroups share the groups of rows, the workgroups of an XCD the units of a group.  An XCD with all of
// its workgroups keeps the weights in registers; with fewer, each takes several blocks of 32 units a step, whose weights it
// fetches every time, and c lives in memory: 128 steps of 64 rows of 1024 units take 0.39 ms with all 256, 2.8 ms with 255, 3.4
// with 100, 34 with 9 (39 ms as soon as one was missing while each went on alone; a launch per step 0.77 ms).  Keeping one block's
// weights in registers there too made that 1.4 ms with 255, and the normal case 6 % slower: half of its fragments then stand
// where the MFMAs have to fetch them from.
// Every result is computed by the same instructions in the same order whoever computes it.
// The control words live where step T-1's projections of batch row 0 begin (scratch); what they displace was saved at the start
// of h_{T-1} (of h_{T-2} where h0 lies there) by the launch before and is fetched into LDS before entering.
#include "igemm_lds.h"

namespace rl {

namespace {

__device__ __forceinline__ void wg_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

constexpr int N_XCD = 8, DEV = 16;              // DEV: cache policy (sc1, device scope) of a load that bypasses the vector L1
// control words: workgroups entered per XCD; ENTERED in all, with CLOSED; PLACED that know their place in their XCD; READY: the entry
// is closed and everyone placed (a cache line of its own: it is what all poll)
constexpr int CTL_ENTERED = N_XCD, CTL_PLACED = N_XCD + 1, CTL_READY = 32, CTL_FLAGS = 64;
constexpr uint32_t CLOSED = 0x80000000u;
constexpr int UNITS = 32;                       // hidden units of a block
constexpr int MAX_POLLS = 1 << 20;              // of a resident workgroup for resident ones: never reached; ends the wait, with NaN in c, all the same

#define RL_CTL_LOAD(i) __hip_atomic_load(ctl + (i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
#define RL_CTL_ADD(i) __hip_atomic_fetch_add(ctl + (i), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)

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
    __shared__ f32x4 part[4][UNITS / 4][64];    // the waves' partial sums
    __shared__ uint32_t saved[CTL_FLAGS + N_XCD * MEMBERS];
    __shared__ uint32_t s_slot;
    __shared__ int s_in;

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int l16 = lane & 15, q4 = lane >> 4;
    uint32_t *ctl = p.ctl;
    const int words = CTL_FLAGS + N_XCD * MEMBERS;
    for (int i = t; i < words; i += 256) saved[i] = p.save[i];
    uint32_t xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    xcc &= N_XCD - 1;
    __syncthreads();                             // the saved words are fetched before this workgroup enters itself

    if (t == 0) {
        s_in = 0;
        const uint32_t before = blockIdx.x < (unsigned)p.let_in ? RL_CTL_ADD(CTL_ENTERED) : CLOSED;
        if (!(before & CLOSED)) {
            s_slot = RL_CTL_ADD(xcc);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // all of this is about the control words alone: their order, no caches
            RL_CTL_ADD(CTL_PLACED);
            const uint64_t begin = wall_clock64();
            auto close = [&]() {
                const uint32_t entered = __hip_atomic_fetch_or(ctl + CTL_ENTERED, CLOSED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (entered & CLOSED) return;
                for (int i = 0; i < MAX_POLLS; ++i)
                    if (RL_CTL_LOAD(CTL_PLACED) == entered) {
                        __hip_atomic_store(ctl + CTL_READY, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        break;
                    }
            };
            if (before + 1 == (uint32_t)p.let_in) close();
            for (int i = 0; i < MAX_POLLS && !s_in; ++i) {
                s_in = (int)RL_CTL_LOAD(CTL_READY);
                const uint64_t waited = wall_clock64() - begin;
                if (s_in || waited < (uint64_t)p.patience) continue;
                const uint32_t entered = RL_CTL_LOAD(CTL_ENTERED);
                if (!(entered & CLOSED) && waited * entered >= (uint64_t)p.patience * (uint32_t)p.let_in) close();
            }
        }
    }
    __syncthreads();
    if (!__builtin_amdgcn_readfirstlane(s_in)) return;
    const int member = __builtin_amdgcn_readfirstlane((int)s_slot);
    const int entered = (int)RL_CTL_LOAD(lane & (N_XCD - 1));   // workgroups of every XCD
    const uint32_t active = (uint32_t)__ballot(entered > 0) & ((1u << N_XCD) - 1);
    const int n_active = __builtin_popcount(active), rank = __builtin_popcount(active & ((1u << xcc) - 1));
    const int members = min(__builtin_amdgcn_readlane(entered, (int)xcc), MEMBERS);
    if (member >= members) return;

    // ---- rows of a group, and what is the same for all of them
    const int R = (p.B + N_XCD - 1) / N_XCD, groups = (p.B + R - 1) / R;      // R at most 16 (checked by the launcher)
    const int N = 4 * H;
    const rsrc_t rw = make_rsrc(p.w, p.w_bytes);
    // packed weight row (= packed column of zx) of (unit, gate)
    auto packed = [](int unit, int gate) { return (unit >> 4) * 64 + gate * 16 + (unit & 15); };
    constexpr int KW = KS / 4, CT = UNITS / 4;
    static_assert(KW % 2 == 0, "a wave takes whole slices of 64");
    auto k_byte = [&](int ks) { return (uint32_t)(((ks >> 1) * 4 + wave) * 128 + (ks & 1) * 64 + q4 * 16); };    // of the lane's part of fragment ks, within a row of H
    auto w_row = [&](int blk, int ct) { return (uint32_t)packed(blk * UNITS + ct * 4 + (l16 >> 2), l16 & 3) * (uint32_t)p.Kp * 2u + (uint32_t)p.k_off * 2u; };
    uint32_t *flags = ctl + CTL_FLAGS + xcc * MEMBERS;
    const rsrc_t rf = make_rsrc(flags, MEMBERS * 4);
    // what a lane finishes: units 4 (2 wave + ct_of(u)) + q4 of a block, of the batch row that lane src_lane has the sums of
    constexpr int NU = HALF ? 1 : 2;
    const int grow = HALF ? l16 & 7 : l16;
    const int src_lane = q4 * 16 + grow;
    auto ct_of = [&](int u) { return HALF ? l16 >> 3 : u; };
    auto unit_of = [&](int blk, int u) { return blk * UNITS + wave * 8 + ct_of(u) * 4 + q4; };
    bool lost = false;
    auto wait_for = [&](uint32_t stamp) {                        // every member's flag says its h is in the L2 (lanes past the members read zero and do not count)
        int i = 0;
#pragma unroll 1
        for (; i < MAX_POLLS; ++i) {
            const uint32_t f = __builtin_amdgcn_raw_buffer_load_b32(rf, (uint32_t)lane * 4u, 0, DEV);
            if (__all(lane >= members || f >= stamp)) break;
            asm volatile("" ::: "memory");
        }
        lost |= i == MAX_POLLS;
    };
    auto publish = [&](uint32_t stamp) {
        // this wave's h is in the L2; after the barrier every wave's is (and every wave has read the partial sums)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        wg_barrier();
        if (t == 0) __hip_atomic_store(flags + member, stamp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto sums = [&](int u) -> f32x4 {
        const int at = wave * 2 + ct_of(u);
        const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
        return (((zero + part[0][at][src_lane]) + part[1][at][src_lane]) + part[2][at][src_lane]) + part[3][at][src_lane];
    };

    uint32_t stamp = 0;                                          // of the last step published
    u32x4 fw[CT][KW];                                            // row l16 = 4 unit + gate of column tile ct, fragment ks of the wave's quarter
    auto multiply = [&](f32x4 (&acc)[CT], const u32x4 (&hf)[KW]) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[ct] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < KW; ++ks)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fw[ct][ks]), __builtin_bit_cast(bf16x8, hf[ks]), acc[ct], 0, 0, 0);
    };
    const bool whole = members == MEMBERS;
    if (whole) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const uint32_t row = w_row(member, ct);
#pragma unroll
            for (int ks = 0; ks < KW; ++ks) fw[ct][ks] = __builtin_amdgcn_raw_buffer_load_b128(rw, row + k_byte(ks), 0, 0);
        }
    }
#pragma unroll 1
    for (int grp = rank; grp < groups && !lost; grp += n_active) {
        const int r0 = grp * R, rows = min(R, p.B - r0);
        const uint32_t h_row = l16 < rows ? (uint32_t)(l16 * ROWB) : 0x80000000u;          // lanes past the rows read zeros
        const bool glive = grow < rows;
        const int row = r0 + min(grow, rows - 1);                // of the units the lane finishes
        auto rsrc_h = [&](int tt) {                              // h_{tt-1} of the group's rows
            const char *src = tt == 0 ? (const char *)p.h0 : (const char *)p.h_seq + (size_t)(tt - 1) * p.h_step_bytes;
            return make_rsrc(src + (size_t)r0 * ROWB, (uint32_t)rows * ROWB);
        };
        auto zx_at = [&](int tt, int unit, int gate) -> float {
            return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(make_rsrc(p.zx + (size_t)tt * p.B * N, (uint32_t)p.B * N * 4u), (uint32_t)(row * N + packed(unit, gate)) * 4u, 0, 0));
        };
        auto zx_true = [&](float z, int tt, int unit, int gate) -> float {       // ... unless the control words stand there
            const int col = packed(unit, gate);
            return tt == p.T - 1 && row == 0 && col < words ? __uint_as_float(saved[col]) : z;
        };
        auto out_row = [&](int tt) { return (uint16_t *)((char *)p.h_seq + (size_t)tt * p.h_step_bytes) + (size_t)row * H; };
        auto bias_at = [&](int unit, int gate) { return p.bias ? p.bias[gate * H + unit] : 0.0f; };
        if (whole) {
            // A wave multiplies all 128 gate columns of the workgroup's block by its quarter of H (its h fragments come straight from
            // the L2 into registers), the quarters meet in LDS, and it finishes eight of the units.
            float bias_r[NU][4], c_r[NU];
#pragma unroll
            for (int u = 0; u < NU; ++u) {
#pragma unroll
                for (int g = 0; g < 4; ++g) bias_r[u][g] = bias_at(unit_of(member, u), g);
                c_r[u] = p.c[(size_t)row * H + unit_of(member, u)];
            }
            float z_r[2][NU][4];                                 // projections of step t and t + 1 (set t & 1)
#pragma unroll
            for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int g = 0; g < 4; ++g) z_r[0][u][g] = zx_at(0, unit_of(member, u), g);
            auto step = [&](int tt, float (&zc)[NU][4], float (&zn)[NU][4]) {
                if (tt > 0) wait_for(stamp);
                const rsrc_t rh = rsrc_h(tt);
                u32x4 hf[KW];
#pragma unroll
                for (int ks = 0; ks < KW; ++ks) hf[ks] = __builtin_amdgcn_raw_buffer_load_b128(rh, h_row + k_byte(ks), 0, DEV);
                __builtin_amdgcn_sched_barrier(0);               // all of them in flight at once; left to itself the compiler asks for two at a time
                const int tn = min(tt + 1, p.T - 1);
#pragma unroll
                for (int u = 0; u < NU; ++u)
#pragma unroll
                    for (int g = 0; g < 4; ++g) zn[u][g] = zx_at(tn, unit_of(member, u), g);
                __builtin_amdgcn_sched_barrier(0);               // the next step's projections are requested here, behind h, and not after the products
                f32x4 acc[CT];
                multiply(acc, hf);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) part[wave][ct][lane] = acc[ct];
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                wg_barrier();
                if (tt == p.T - 1 && r0 == 0) {
#pragma unroll
                    for (int u = 0; u < NU; ++u)
#pragma unroll
                        for (int g = 0; g < 4; ++g) zc[u][g] = zx_true(zc[u][g], tt, unit_of(member, u), g);
                }
                uint16_t *out = out_row(tt);
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const f32x4 a = sums(u);
                    float z[4];
#pragma unroll
                    for (int g = 0; g < 4; ++g) z[g] = (a[g] + zc[u][g]) + bias_r[u][g];
                    const float hn = lstm_cell_(z, c_r[u]);
                    if (glive) out[unit_of(member, u)] = (uint16_t)f32_to_bf16_bits(hn);
                }
                publish(++stamp);
            };
#pragma unroll 1
            for (int tt = 0; tt < p.T; tt += 2) {
                step(tt, z_r[0], z_r[1]);
                if (tt + 1 < p.T) step(tt + 1, z_r[1], z_r[0]);
                if (lost) break;
            }
#pragma unroll
            for (int u = 0; u < NU; ++u)
                if (glive) p.c[(size_t)row * H + unit_of(member, u)] = lost ? __uint_as_float(0x7fc00000u) : c_r[u];
        } else {
            // fewer workgroups than blocks of units: the same block after block, the weights fetched every time,
            // one column tile ahead of the products
#pragma unroll 1
            for (int tt = 0; tt < p.T && !lost; ++tt) {
                if (tt > 0) wait_for(stamp);
                const rsrc_t rh = rsrc_h(tt);
                u32x4 hf[KW];
#pragma unroll
                for (int ks = 0; ks < KW; ++ks) hf[ks] = __builtin_amdgcn_raw_buffer_load_b128(rh, h_row + k_byte(ks), 0, DEV);
#pragma unroll 1
                for (int blk = member; blk < MEMBERS; blk += members) {
                    f32x4 acc[CT];
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) acc[ct] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    u32x4 fs[2][KW];
                    auto fetch = [&](int ct) {
#pragma unroll
                        for (int ks = 0; ks < KW; ++ks) fs[ct & 1][ks] = __builtin_amdgcn_raw_buffer_load_b128(rw, w_row(blk, ct) + k_byte(ks), 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    fetch(0);
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        if (ct + 1 < CT) fetch(ct + 1);
#pragma unroll
                        for (int ks = 0; ks < KW; ++ks)
                            acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fs[ct & 1][ks]), __builtin_bit_cast(bf16x8, hf[ks]), acc[ct], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (blk != member) wg_barrier();             // the block before is read out
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) part[wave][ct][lane] = acc[ct];
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    wg_barrier();
#pragma unroll
                    for (int u = 0; u < NU; ++u) {
                        const int unit = unit_of(blk, u);
                        const f32x4 a = sums(u);
                        float z[4];
#pragma unroll
                        for (int g = 0; g < 4; ++g) z[g] = (a[g] + zx_true(zx_at(tt, unit, g), tt, unit, g)) + bias_at(unit, g);
                        float *cp = p.c + (size_t)row * H + unit;
                        float c = *cp;
                        const float hn = lstm_cell_(z, c);
                        if (glive) {
                            *cp = c;
                            out_row(tt)[unit] = (uint16_t)f32_to_bf16_bits(hn);
                        }
                    }
                }
                publish(++stamp);
            }
            if (lost && glive)
                for (int blk = member; blk < MEMBERS; blk += members)
#pragma unroll
                    for (int u = 0; u < NU; ++u) p.c[(size_t)row * H + unit_of(blk, u)] = __uint_as_float(0x7fc00000u);
        }
    }
#endif
}

#define RL_INST(KS) template __global__ void lstm_seq_kernel<KS, false>(const LstmSeqParams); template __global__ void lstm_seq_kernel<KS, true>(const LstmSeqParams);
RL_INST(8) RL_INST(16) RL_INST(24) RL_INST(32)
#undef RL_INST

// From 16 steps on, or 12 where a step's own launch (H / 8 x B / 32 workgroups) does not fit on the 256 CUs at once: entering and
// fetching the weights take as long as 8 to 10 steps.  Step by step / in one launch, us with the projections: 16 steps of 1 x 1024
// units 84 / 77, 64 x 1024 98 / 94, 64 x 256 76 / 58; 12 steps 65 / 73, 77 / 87, 58 / 54, of 128 x 768 103 / 90; 8 steps 45 / 66,
// 57 / 76, 41 / 50, 72 / 78.
bool lstm_seq_ok(int64_t B, int64_t H, int64_t T)
{
    return B >= 1 && B <= 16 * N_XCD && H >= 256 && H <= 1024 && H % 256 == 0 && T >= (H / 8 * ((B + 31) / 32) > 256 ? 12 : 16);
}

// A stream that was given a part of the CUs gets the launches of a step each: a cooperative launch goes out on a queue of its own,
// which need not keep to that part.
static bool whole_device(hipStream_t s)
{
    uint32_t mask[32] = {0};
    if (hipExtStreamGetCUMask(s, 32, mask) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    int dev = 0, cus = 0, set = 0;
    for (uint32_t m : mask) set += __builtin_popcount(m);
    return hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || set >= cus;
}

hipError_t launch_lstm_seq(const LstmSeqParams &p0, hipStream_t s)
{
    LstmSeqParams p = p0;
    if (!lstm_seq_ok(p.B, p.H, p.T) || !p.h0 || !p.h_seq || !p.w || !p.zx || !p.c || !p.ctl || !p.save || p.let_in < 0 || p.patience < 0 || p.Kp < p.k_off + p.H || p.k_off < 0 || p.k_off % 8 != 0 ||
        p.Kp % 8 != 0 || (uint64_t)4 * p.H * p.Kp * 2 != p.w_bytes || p.w_bytes >= 0x7fffffffu || p.h_step_bytes < (size_t)p.B * p.H * 2 ||
        ((uintptr_t)p.ctl & 255) || ((uintptr_t)p.save & 3))
        return hipErrorInvalidValue;
    if (!whole_device(s)) return hipErrorNotSupported;
    static const void *const kerns[4][2] = {{(const void *)lstm_seq_kernel<8, false>, (const void *)lstm_seq_kernel<8, true>}, {(const void *)lstm_seq_kernel<16, false>, (const void *)lstm_seq_kernel<16, true>},
                                            {(const void *)lstm_seq_kernel<24, false>, (const void *)lstm_seq_kernel<24, true>}, {(const void *)lstm_seq_kernel<32, false>, (const void *)lstm_seq_kernel<32, true>}};
    const void *kern = kerns[p.H / 256 - 1][p.B <= 8 * N_XCD];
    const int grid = N_XCD * (p.H / UNITS);
    p.let_in = p.let_in == 0 || p.let_in > grid ? grid : p.let_in;
    hipLaunchKernelGGL(lstm_seq_prepare_kernel, dim3(1), dim3(256), 0, s, p.ctl, p.save, lstm_seq_ctl_words(p.H), 0);
    hipError_t er = hipGetLastError();
    if (er != hipSuccess) return er;
    void *args[] = {&p};
    er = hipLaunchCooperativeKernel(kern, dim3((unsigned)grid), dim3(256), args, 0, s);
    if (er == hipSuccess) return er;
    // this device cannot hold the grid (or has no cooperative launches): the projections as they were, for the caller's other form
    (void)hipGetLastError();
    hipLaunchKernelGGL(lstm_seq_prepare_kernel, dim3(1), dim3(256), 0, s, p.ctl, p.save, lstm_seq_ctl_words(p.H), 1);
    (void)hipGetLastError();
    return hipErrorNotSupported;
}

}  // namespace rl
