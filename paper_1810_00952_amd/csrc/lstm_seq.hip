// A whole LSTM sequence in one launch, input projections already done (zx of every step, packed column order):
//
//   z_t = zx_t + h_{t-1} . Wh^T + bias;  c_t, h_t by the gates (see lstm_step.hip)
//
// What bounds the one-launch-per-step form is not its arithmetic: 6.3 us per step, of which about 3 pass between dependent
// launches and the rest fetching 128 KB per CU again (64 KB of weights that never change).  Here every CU keeps its weights in
// registers for the whole sequence and a step costs one exchange of h between the CUs that need it: about 1.6 us at 64 rows of
// 1024 units (128 steps with their projections: 814 us step by step, 303 us here, 79 of them the projections).  What is left of a
// step is a chain: the L2 round trip for h (900 cycles), the products (1050, half of the MFMA's columns empty), the partial sums
// through LDS (350), the gates (600), the way of the result to the L2.

// Split: batch rows over the eight XCDs (8 of 64), hidden units over the CUs of an XCD (32 each at H = 1024).  Inside a CU each
// of the four waves multiplies all 128 gate columns by its quarter of H (256 registers of weights per lane at H = 1024), so that
// h is fetched once per CU, each wave its own part straight into registers; the four partial sums meet in LDS.  Wave w's quarter
// are the slices w, w + 4, ... of 64 contraction indices, summed and added up in the order of lstm_step.hip: the two forms give
// the same bits, so that which of them runs a sequence is a matter of time alone.  (Eight units
// per wave over the whole of H, with h staged in LDS: 520 us.  Quarters with the loads left to the compiler, which asks for h two
// fragments at a time and for the projections only after the products: 548 us.)
// A step's h is written and read inside one XCD, through its L2: the stores go there (the vector L1 writes through), the loads
// bypass the L1 (device scope; the narrower scopes may hit it).  No cache is flushed, which is what made a grid-wide barrier
// cost more than a launch.
// The members of a group exchange h in a ring of four steps, in the order of the MFMA fragments, apart from the results: its lines
// stay in the L2, a wave writes whole lines and reads 512 or 1024 bytes in a row.  (Read from the results themselves, a step's h took
// 2700 cycles to come: 32 loads of scattered rows at 50 cycles each, of lines that the L2 had only parts of.)  The ring lies where
// the group's projections of step 0 were.  Its words say themselves that they are there: every wave clears its words of the next
// step to NOT_YET, which no h is, under the products, before it writes this step's, and a reader asks again until none is left; who
// has seen all of step t - 1 knows everyone past step t - 2, so that nobody still reads the words that are cleared.  The first steps
// go by flags: a workgroup publishes step t by writing t + 1 into its flag word after its stores were acknowledged, and the members
// poll the flags of all of them (every step that way: 391 us with a row-major ring, 405 through the results).
// What else the step's chain lost: stores of results and of cleared words, and the requests for projections, go out one at a time between the
// products (all at once 306 us), the first steps are code of their own (327 -> 313), sums and lane moves stay out of AGPRs (-> 305).
// MFMA 16x16x32, weights as the row operand with row 4u + gate: a lane's four result registers are the four gates of one
// (unit, batch row), so the gates, c (in registers throughout) and h need no exchange between lanes.
//
// Waiting for other workgroups is safe only if they are resident.  So a workgroup first enters itself in the control block, and
// the first one to see all of them there closes the entry, or the first one that has waited longer than the sequence would take
// the workgroups that are there (3 us a step at full strength): they wait for no one else, whoever starts later returns at once.
// The XCDs that have workgroups share the groups of rows, the workgroups of an XCD the units of a group.  An XCD with all of
// its workgroups keeps the weights in registers; with fewer, each takes several blocks of 32 units a step, whose weights it
// fetches every time, and c lives in memory: 128 steps of 64 rows of 1024 units take 0.30 ms with all 256, 2.8 ms with 255, 3.4
// with 100, 34 with 9 (39 ms as soon as one was missing while each went on alone; a launch per step 0.77 ms).  Keeping one block's
// weights in registers there too made that 1.4 ms with 255, and the normal case 6 % slower: half of its fragments then stand
// where the MFMAs have to fetch them from.
// Every result is computed by the same instructions in the same order whoever computes it.
// The control words live where step T-1's projections of batch row 0 begin (scratch); what they displace was saved at the start
// of h_{T-1} (of h_{T-2} where h0 lies there) by the launch before and is fetched into LDS before entering.
#include <type_traits>

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
// Steps from this one on wait for the words of h themselves, cleared to NOT_YET (infinity and zero; |h| is 1 at most, or NaN) a step ahead;
// the earlier ones for the flags (h0 may lie in any slot but the first, and is read until everyone has published step 0)
constexpr int BY_WORD = 3;
constexpr uint32_t NOT_YET = 0x7f800000u;
constexpr int ROR8 = 0x128;                       // DPP: a row of sixteen lanes rotated by eight
constexpr int RING = 4;                         // steps of h the exchange holds
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
// every other unit in the gate arithmetic, which is a serial chain of exponentials (128 steps of 64 rows, projections in cache: 498 -> 446 us),
// and the odd one of two column tiles, or of two fragments of h.
template <int KS, bool HALF>
__global__ __launch_bounds__(256, 1) void lstm_seq_kernel(const LstmSeqParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub; the body uses gfx950-only builtins
    constexpr int H = KS * 32, MEMBERS = H / UNITS, ROWB = H * 2;
    __shared__ f32x4 part[2][4][UNITS / 4][64]; // the waves' partial sums; of even and odd steps where a step has one barrier
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
        const bool may_enter = p.xcds < N_XCD ? (int)(blockIdx.x % N_XCD) < p.xcds : blockIdx.x < (unsigned)p.let_in;
        const uint32_t before = may_enter ? RL_CTL_ADD(CTL_ENTERED) : CLOSED;
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
        // this wave's h is in the L2; after the barrier every wave's is
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        wg_barrier();
        if (t == 0) __hip_atomic_store(flags + member, stamp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto sums = [&](int u) -> f32x4 {
        const int at = wave * 2 + ct_of(u);
        const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
        return (((zero + part[0][0][at][src_lane]) + part[0][1][at][src_lane]) + part[0][2][at][src_lane]) + part[0][3][at][src_lane];
    };
    // The words of a row of h that a lane writes and clears, two units each: units 4 ct + (q4 & ~1) and the one behind it.  Sixteen rows
    // a group: a lane has two units of its own (ct 0 and 1) and trades one with the lane 16 further; eight rows: the even q4 write.
    const bool writes = !HALF || !(q4 & 1);
    const int word_unit = wave * 8 + (HALF ? l16 >> 3 : q4 & 1) * 4 + (q4 & 2);
    auto two_units = [&](const uint32_t (&h)[NU]) -> uint32_t {
        const auto r = __builtin_amdgcn_permlane16_swap(h[0], h[NU - 1], false, false);      // odd rows of 16 lanes of the first against the even ones of the second
        return r[0] | r[1] << 16;
    };

    uint32_t stamp = 0;                                          // of the last step published
    u32x4 fw[CT][KW];                                            // row l16 = 4 unit + gate of column tile ct, fragment ks of the wave's quarter
    auto multiply = [&](f32x4 (&acc)[CT], auto h_of, auto meanwhile) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[ct] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < KW; ++ks) {
            const u32x4 h = h_of(ks);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fw[ct][ks]), __builtin_bit_cast(bf16x8, h), acc[ct], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            meanwhile(ks);
            __builtin_amdgcn_sched_barrier(0);
        }
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
            // The members' exchange of h (steps from BY_WORD on): a few steps' worth where step 0's projections of the group's rows were, so
            // that the lines stay in the L2, in the order of the fragments: [fragment = member][quarter = wave][row][8 units].
            // A wave writes whole lines and reads a KB at a time.  With at most eight rows the lanes of the other eight columns fetch
            // the fragment behind.
            constexpr int NL = HALF ? KW / 2 : KW;
            const uint32_t slot = (uint32_t)rows * ROWB;
            const rsrc_t rr = make_rsrc(p.zx + (size_t)r0 * N, RING * slot);
            auto ring = [&](int tt) { return (uint32_t)(tt % RING) * slot; };
            const uint32_t word_at = writes && glive ? (uint32_t)(((member * 4 + wave) * rows + grow) * 16 + (word_unit & 7) * 2) : OOB;
            const uint32_t out_at = writes && glive ? (uint32_t)(row * ROWB + (member * UNITS + word_unit) * 2) : OOB;
            const uint32_t ring_at = glive ? (uint32_t)((((HALF ? l16 >> 3 : 0) * 4 + q4) * rows + grow) * 16) : OOB;
            const uint32_t seq_at = glive ? (uint32_t)(grow * ROWB + (HALF ? l16 >> 3 : 0) * 64 + q4 * 16) : OOB;
            uint32_t word = 0;                                   // what the lane writes of a step's h
            auto write_out = [&](int tt) {
                __builtin_amdgcn_raw_buffer_store_b32(word, make_rsrc((char *)p.h_seq + (size_t)tt * p.h_step_bytes, (uint32_t)p.B * ROWB), out_at, 0, 0);
            };
            auto step = [&](auto phase, int tt, float (&zc)[NU][4], float (&zn)[NU][4]) {
                constexpr bool by_word = decltype(phase)::value;
                if (tt > 0 && !by_word) wait_for(stamp);
                u32x4 hl[NL];
                const rsrc_t rh = by_word ? rr : rsrc_h(tt);
                const uint32_t at = by_word ? ring_at : seq_at, base = by_word ? ring(tt - 1) : 0u, unit = by_word ? (uint32_t)rows * 128u : 128u;
                auto fetch = [&]() {
#pragma unroll
                    for (int i = 0; i < NL; ++i) {
                        const int ks = HALF ? 2 * i : i;         // slice (ks >> 1) * 4 + wave, two fragments
                        hl[i] = __builtin_amdgcn_raw_buffer_load_b128(rh, at, base + (uint32_t)((ks >> 1) * 4 + wave) * unit + ((ks & 1) ? unit / 2 : 0u), DEV);
                    }
                    __builtin_amdgcn_sched_barrier(0);           // all of them in flight at once; left to itself the compiler asks for two at a time
                };
                fetch();
                if (by_word) {
                    int i = 0;
#pragma unroll 1
                    for (; i < MAX_POLLS; ++i) {
                        float top = -2.0f;                       // of the words as numbers; a NaN in a word does not count
#pragma unroll
                        for (int i = 0; i < NL; ++i) {
                            asm("v_max3_f32 %0, %1, %2, %0" : "+v"(top) : "v"(hl[i][0]), "v"(hl[i][1]));
                            asm("v_max3_f32 %0, %1, %2, %0" : "+v"(top) : "v"(hl[i][2]), "v"(hl[i][3]));
                        }
                        if (__all(top < 2.0f)) break;
                        asm volatile("" ::: "memory");
                        fetch();
                    }
                    lost |= i == MAX_POLLS;
                }
                f32x4 acc[CT];
                multiply(acc, [&](int ks) {
                    if constexpr (!HALF) return hl[ks];
                    u32x4 v = hl[ks >> 1];
                    if (ks & 1) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = (uint32_t)__builtin_amdgcn_mov_dpp((int)v[e], ROR8, 0xf, 0xf, false);      // from eight lanes on in the row of sixteen
                    }
                    return v;
                }, [&](int ks) {
                    // under the products, a request at a time: the step before's h into the results, the words of the next one cleared, the
                    // next step's projections
                    constexpr int OPS = 2 + 4 * NU;
#pragma unroll
                    for (int i = ks * OPS / KW; i < (ks + 1) * OPS / KW; ++i) {
                        if (i == 0) {
                            if (by_word) write_out(tt - 1);
                        } else if (i == 1) {
                            if (by_word || tt >= BY_WORD - 2) __builtin_amdgcn_raw_buffer_store_b32(NOT_YET, rr, word_at, ring(tt + 1), 0);
                            __builtin_amdgcn_sched_barrier(0);   // ahead of every load below: the wait before the step's words counts on that
                        } else {
                            zn[(i - 2) / 4][(i - 2) % 4] = zx_at(min(tt + 1, p.T - 1), unit_of(member, (i - 2) / 4), (i - 2) % 4);
                        }
                    }
                });
                f32x4 (&sums_of)[4][UNITS / 4][64] = part[tt & 1];
                if constexpr (HALF) {
                    // eight columns of a tile are empty: two tiles a register, the odd one in the upper eight lanes, where it is finished
#pragma unroll
                    for (int ct = 0; ct < CT; ct += 2) {
                        f32x4 v;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            v[e] = __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(acc[ct][e]), __float_as_int(acc[ct + 1][e]), ROR8, 0xf, 0xc, false));
                        sums_of[wave][ct >> 1][lane] = v;
                    }
                } else {
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) sums_of[wave][ct][lane] = acc[ct];
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                wg_barrier();
                if (tt == p.T - 1 && r0 == 0) {
#pragma unroll
                    for (int u = 0; u < NU; ++u)
#pragma unroll
                        for (int g = 0; g < 4; ++g) zc[u][g] = zx_true(zc[u][g], tt, unit_of(member, u), g);
                }
                uint32_t hb[NU];
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int at = HALF ? wave : wave * 2 + u;
                    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
                    const f32x4 a = (((zero + sums_of[0][at][lane]) + sums_of[1][at][lane]) + sums_of[2][at][lane]) + sums_of[3][at][lane];
                    float z[4];
#pragma unroll
                    for (int g = 0; g < 4; ++g) z[g] = (a[g] + zc[u][g]) + bias_r[u][g];
                    const uint32_t h = __float_as_uint(lstm_cell_(z, c_r[u])), up = (h + 0x7fffu + (h >> 16 & 1u)) >> 16, nan = h >> 16 | 0x40u;      // f32_to_bf16_bits without a branch
                    hb[u] = (h & 0x7fffffffu) > 0x7f800000u ? nan : up;
                }
                word = two_units(hb);
                // the next step's words are cleared before this step's are written: the 4 NU loads of projections behind the clearing store may be
                // on their way still, it may not
                asm volatile("s_waitcnt vmcnt(%0)" :: "n"(4 * NU) : "memory");
                if (by_word || tt >= BY_WORD - 1) __builtin_amdgcn_raw_buffer_store_b32(word, rr, word_at, ring(tt), 0);
                else write_out(tt);
                if (!by_word && tt + 1 < BY_WORD) publish(++stamp);
            };
            static_assert(BY_WORD == 3, "written out here");     // T is 12 at least
            step(std::false_type{}, 0, z_r[0], z_r[1]);
            step(std::false_type{}, 1, z_r[1], z_r[0]);
            step(std::false_type{}, 2, z_r[0], z_r[1]);
#pragma unroll 1
            for (int tt = BY_WORD; tt < p.T && !lost; tt += 2) {
                step(std::true_type{}, tt, z_r[1], z_r[0]);
                if (tt + 1 < p.T) step(std::true_type{}, tt + 1, z_r[0], z_r[1]);
            }
            write_out(p.T - 1);
#pragma unroll
            for (int u = 0; u < NU; ++u)
                if (glive) p.c[(size_t)row * H + unit_of(member, u)] = lost ? __uint_as_float(0x7fc00000u) : c_r[u];
            // the last step's sums are read out before the next group's first step writes there: with an odd number of steps both are part[0]
            if (grp + n_active < groups) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                wg_barrier();
            }
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
                    for (int ct = 0; ct < CT; ++ct) part[0][wave][ct][lane] = acc[ct];
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
    if (!lstm_seq_ok(p.B, p.H, p.T) || !p.h0 || !p.h_seq || !p.w || !p.zx || !p.c || !p.ctl || !p.save || p.let_in < 0 || p.xcds < 0 || p.patience < 0 || p.Kp < p.k_off + p.H || p.k_off < 0 || p.k_off % 8 != 0 ||
        p.Kp % 8 != 0 || (uint64_t)4 * p.H * p.Kp * 2 != p.w_bytes || p.w_bytes >= 0x7fffffffu || p.h_step_bytes < (size_t)p.B * p.H * 2 ||
        ((uintptr_t)p.ctl & 255) || ((uintptr_t)p.save & 3))
        return hipErrorInvalidValue;
    if (!whole_device(s)) return hipErrorNotSupported;
    static const void *const kerns[4][2] = {{(const void *)lstm_seq_kernel<8, false>, (const void *)lstm_seq_kernel<8, true>}, {(const void *)lstm_seq_kernel<16, false>, (const void *)lstm_seq_kernel<16, true>},
                                            {(const void *)lstm_seq_kernel<24, false>, (const void *)lstm_seq_kernel<24, true>}, {(const void *)lstm_seq_kernel<32, false>, (const void *)lstm_seq_kernel<32, true>}};
    const void *kern = kerns[p.H / 256 - 1][p.B <= 8 * N_XCD];
    const int grid = N_XCD * (p.H / UNITS);
    p.let_in = p.let_in == 0 || p.let_in > grid ? grid : p.let_in;
    p.xcds = p.xcds == 0 || p.xcds > N_XCD ? N_XCD : p.xcds;
    if (p.xcds < N_XCD) p.let_in = p.xcds * (p.H / UNITS);
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
