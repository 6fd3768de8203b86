// Fusion-group planner and executor (host).
//
// For every caller-declared group the planner re-checks legality, picks the
// kernel (implicit-GEMM contraction with epilogue, single-pass elementwise
// chain, window reduction, gate kernel), the tile, and the private layout of
// each intermediate: rank-4 activations between contractions live
// channel-last so that a K slice of the implicit GEMM is a run of channels;
// tensors at the boundary keep the order of their Shape.  Layout changes are
// inserted only where a consumer cannot read what its producer wrote.
#include "plan.h"

#include <algorithm>
#include <cmath>
#include <set>
#include <sstream>

namespace rl {

namespace {

enum { L_NATIVE = 0, L_NHWC = 1 };

inline int64_t round_up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }
inline int kv_of(int dtype) { return dtype == RL_BF16 ? 8 : 4; }

// a change of layout without its pointers
MoveParams move_params(const Step &t)
{
    MoveParams m{nullptr, nullptr, t.t_dtype, t.t_N, t.t_C, t.t_P, t.kind == S_PAD_NHWC ? t.st_W : 0};
    if (t.kind == S_TO_NCHW) std::swap(m.R, m.Q);
    return m;
}

struct Planner {
    const Graph &g;
    Plan &plan;
    std::string &msg;
    std::vector<int> phys[2];              // [layout][value] -> buffer index or -1
    std::set<int> out_set;
    std::vector<std::vector<int>> consumers;
    std::map<int, int> padded_rows;        // value -> buffer of its channels-fastest rows padded to whole 16-byte vectors

    Planner(const Graph &g_, Plan &p_, std::string &m_) : g(g_), plan(p_), msg(m_) {}

    rl_status fail(rl_status st, const std::string &m) { msg = m; return st; }

    const rl_type &T(int v) const { return g.values[v].type; }
    bool hw1(int v) const { return T(v).rank == 4 && T(v).dims[2] * T(v).dims[3] == 1; }
    bool layout_free(int v) const { return T(v).rank != 4 || hw1(v) || T(v).dims[1] == 1; }
    size_t bytes_of(int v) const { return (size_t)numel(T(v)) * dtype_size(T(v).dtype); }

    int bound(int v)
    {
        if (plan.bound_buf[v] < 0) {
            BufDesc b;
            b.bound_value = v;
            b.bytes = bytes_of(v);
            plan.bufs.push_back(b);
            plan.bound_buf[v] = (int)plan.bufs.size() - 1;
        }
        return plan.bound_buf[v];
    }
    int new_ws(size_t bytes)
    {
        BufDesc b;
        b.bytes = round_up((int64_t)bytes, 256);
        plan.bufs.push_back(b);
        return (int)plan.bufs.size() - 1;
    }
    void set_phys(int v, int layout, int buf)
    {
        phys[layout][v] = buf;
        if (layout_free(v)) phys[1 - layout][v] = buf;
    }
    // A graph output that is the channel-last view (layout_transform with axes 0,2,3,1) of rank-4 value v, or -1:
    // v's channel-last storage then is that output's own buffer.
    int channel_last_output_of(int v) const
    {
        for (int c : consumers[v]) {
            const OpNode &o = g.ops[c];
            if (o.kind == RL_OP_LAYOUT_TRANSFORM && T(v).rank == 4 && o.attrs.perm[0] == 0 && o.attrs.perm[1] == 2 && o.attrs.perm[2] == 3 &&
                o.attrs.perm[3] == 1 && out_set.count(o.out[0]))
                return o.out[0];
        }
        return -1;
    }
    // buffer a step writes value v into, in `layout`
    int out_buf(int v, int layout)
    {
        int b, home;
        if (out_set.count(v) && (layout == L_NATIVE || layout_free(v))) b = bound(v);
        else if (layout == L_NHWC && !layout_free(v) && (home = channel_last_output_of(v)) >= 0) b = bound(home);
        else b = new_ws(bytes_of(v));
        set_phys(v, layout, b);
        return b;
    }
    Step &add_step(int kind, const std::string &name, const std::string &kernel)
    {
        plan.steps.emplace_back();
        Step &s = plan.steps.back();
        s.kind = kind;
        s.name = name;
        s.kernel = kernel;
        return s;
    }
    // make value v available in `layout`; returns the buffer
    rl_status need(int v, int layout, int &buf)
    {
        if (phys[layout][v] >= 0) { buf = phys[layout][v]; return RL_OK; }
        int other = phys[1 - layout][v];
        if (other < 0) return fail(RL_ERR_UNSUPPORTED, "internal: value has no storage yet");
        const rl_type &t = T(v);
        int dst = out_buf(v, layout);
        Step &s = add_step(layout == L_NHWC ? S_TO_NHWC : S_TO_NCHW, "layout", layout == L_NHWC ? "nchw_to_nhwc" : "nhwc_to_nchw");
        s.t_dtype = t.dtype; s.t_N = (int)t.dims[0]; s.t_C = (int)t.dims[1]; s.t_P = (int)(t.dims[2] * t.dims[3]);
        s.slot[SL_X] = other; s.slot[SL_Y] = dst;
        s.bytes = 2.0 * bytes_of(v);
        buf = dst;
        return RL_OK;
    }

    // ---- injective chain -------------------------------------------------
    struct Chain {
        Epilogue epi{};
        std::vector<int> operand;        // value id per pointer slot
        std::vector<bool> is_vec;        // bias vector (1-D) or full-shape tensor
        int bias_axis = -1;
        int last_value = -1;
    };
    rl_status push_op(Chain &c, uint8_t op, int operand, bool vec)
    {
        if (c.epi.n_ops >= RL_EPI_MAX_OPS) return fail(RL_ERR_UNSUPPORTED, "fused chain longer than the kernel's program");
        int a = 0;
        if (operand >= 0) {
            a = -1;
            for (size_t i = 0; i < c.operand.size(); ++i)
                if (c.operand[i] == operand) a = (int)i;
            if (a < 0) {
                if ((int)c.operand.size() >= RL_EPI_MAX_PTRS) return fail(RL_ERR_UNSUPPORTED, "fused chain has too many operands");
                c.operand.push_back(operand);
                c.is_vec.push_back(vec);
                a = (int)c.operand.size() - 1;
                epi_set_dtype(c.epi, a, T(operand).dtype);
            }
        }
        epi_set_op(c.epi, c.epi.n_ops, op, a);
        c.epi.n_ops++;
        return RL_OK;
    }
    // ops[from..to) applied to running value `cur`
    rl_status build_chain(const std::vector<int> &ops, size_t from, size_t to, int cur, const std::set<int> &gset, Chain &c)
    {
        for (size_t i = from; i < to; ++i) {
            const OpNode &o = g.ops[ops[i]];
            auto external = [&](int v) { return g.values[v].producer < 0 || !gset.count(g.values[v].producer); };
            rl_status st = RL_OK;
            switch (o.kind) {
            case RL_OP_NEG: case RL_OP_SQ: case RL_OP_RELU: case RL_OP_SIGMOID: case RL_OP_TANH: case RL_OP_CAST: {
                if (o.in[0] != cur) return fail(RL_ERR_UNSUPPORTED, "fused group is not a single chain");
                uint8_t code = o.kind == RL_OP_NEG ? E_NEG : o.kind == RL_OP_SQ ? E_SQ : o.kind == RL_OP_RELU ? E_RELU
                             : o.kind == RL_OP_SIGMOID ? E_SIGMOID : o.kind == RL_OP_TANH ? E_TANH
                             : (o.attrs.to == RL_BF16 ? E_ROUND_BF16 : E_NOP);
                st = push_op(c, code, -1, false);
                break;
            }
            case RL_OP_BIAS_ADD:
                if (o.in[0] != cur || !external(o.in[1])) return fail(RL_ERR_UNSUPPORTED, "fused group is not a single chain");
                if (c.bias_axis >= 0 && c.bias_axis != o.attrs.axis) return fail(RL_ERR_UNSUPPORTED, "bias_add along two axes in one group");
                c.bias_axis = o.attrs.axis;
                st = push_op(c, E_BIAS, o.in[1], true);
                break;
            case RL_OP_ADD: case RL_OP_SUB: case RL_OP_MUL: case RL_OP_DIV: {
                int a = o.in[0], b = o.in[1];
                if (a == cur && b == cur) {
                    uint8_t code = o.kind == RL_OP_ADD ? E_ADD_VV : o.kind == RL_OP_SUB ? E_SUB_VV : o.kind == RL_OP_MUL ? E_SQ : E_DIV_VV;
                    st = push_op(c, code, -1, false);
                } else if (a == cur && external(b)) {
                    uint8_t code = o.kind == RL_OP_ADD ? E_ADD : o.kind == RL_OP_SUB ? E_SUB : o.kind == RL_OP_MUL ? E_MUL : E_DIV;
                    st = push_op(c, code, b, false);
                } else if (b == cur && external(a)) {
                    uint8_t code = o.kind == RL_OP_ADD ? E_ADD : o.kind == RL_OP_SUB ? E_RSUB : o.kind == RL_OP_MUL ? E_MUL : E_RDIV;
                    st = push_op(c, code, a, false);
                } else {
                    return fail(RL_ERR_UNSUPPORTED, "fused group is not a single chain");
                }
                break;
            }
            default:
                return fail(RL_ERR_UNSUPPORTED, std::string(op_name(o.kind)) + " inside a chain");
            }
            if (st != RL_OK) return st;
            cur = o.out[0];
        }
        c.last_value = cur;
        return RL_OK;
    }
    // bind the chain's operands to step slots; full-shape operands in `layout`
    rl_status bind_chain(Chain &c, Step &s, int layout, double &bytes)
    {
        for (size_t i = 0; i < c.operand.size(); ++i) {
            int buf;
            rl_status st = need(c.operand[i], c.is_vec[i] ? L_NATIVE : layout, buf);
            if (st != RL_OK) return st;
            // `need` may have appended a layout step: s is re-fetched by the caller, so only indices are kept here
            s.slot[SL_E0 + i] = buf;
            bytes += (double)bytes_of(c.operand[i]);
        }
        return RL_OK;
    }

    // ---- contraction groups ------------------------------------------------
    // A contraction seen through other eyes than its op's: the gradient with respect to the first operand of a dense
    // or of a stride-1 conv2d is a dense / a stride-1 conv2d of dy with re-ordered weights, and runs on the same kernels.
    struct AnchorView {
        int kind;                         // RL_OP_DENSE or RL_OP_CONV2D
        int N, KH, KW, ph, pw;            // output channels (features), taps, padding; stride 1; contraction channels come from x
        GatherPack gp;                    // where the rows of the K-contiguous weight matrix come from
        int xbuf = -1;                    // >= 0: the activations are this channel-last buffer [xN][xH][xW][C] instead of x's own
        int xH = 0, xW = 0, xC = 0;       // xC: channels of a pixel there, zeros behind x's own (0: as many as x has)
    };

    // Shader cycles per K tile of the direct-load kernel on the fullest of 256 CUs: `alone` where a CU holds one workgroup, `share`
    // per workgroup where it holds several (measured; f32 is the MFMA's own 1024 / 2048 / 4096 and a few percent).  Of four waves, as K slices and
    // larger grids run: whole grids of up to 256 workgroups of 64x64 tiles run eight (TEAMS in igemm_dma.h) and take 0.95 to 0.99 of it
    static double tile_cost(int tile, int dtype, int64_t workgroups)
    {
        static const double alone[2][3] = {{4400, 2300, 1450}, {1400, 900, 680}}, share[2][3] = {{4400, 2100, 1100}, {1200, 600, 390}};
        const int d = dtype == RL_BF16;
        return std::max(alone[d][tile], share[d][tile] * (double)((workgroups + 255) / 256));
    }
    // 128x64 or 64x64 tiles, by the padding of the last ones and how the grid fills 256 CUs; the f32 MFMA takes so long that small
    // tiles cost nothing where they fill the chip better (16x128x28x28 -> 128 3x3: 128x64 67.8 us, 64x64 47.7)
    // (never 128x128: f32 has no gain from it, and bf16 across taps holds one such workgroup per CU; 48 layers that took it ran
    // in 0.87 of its time on 128x64)
    static int direct_load_tile(int dtype, int64_t M, int64_t N)
    {
        auto cost = [&](int tile, int64_t bm) { return tile_cost(tile, dtype, ((M + bm - 1) / bm) * ((N + 63) / 64)); };
        return cost(TILE_64x64, 64) < cost(TILE_128x64, 128) ? TILE_64x64 : TILE_128x64;
    }

    // Few tiles and a long K (small batches, late stages): K is split over several workgroups per tile, whose fp32
    // sums meet in a scratch tensor [splits][M][N] that a second kernel adds up in order before the epilogue.
    // splits = 1: whole; per: K tiles of a slice; cycles: of the fullest CU, the adding launch's share included (up to 64 tiles with the
    // slices that each gain a twentieth; direct_form's constants are fitted to that)
    struct KSlices { int splits = 1, per = 0; int64_t tiles = 0; double cycles = 0.0; };
    KSlices k_slices(int tile, int dtype, int64_t M, int64_t N, int64_t K) const
    {
        static const int tbm[] = {128, 128, 64}, tbn[] = {128, 64, 64};
        const int BK = 8 * kv_of(dtype), nk = (int)((K + BK - 1) / BK);
        KSlices c;
        c.tiles = ((M + tbm[tile] - 1) / tbm[tile]) * ((N + tbn[tile] - 1) / tbn[tile]);
        c.per = nk;
        c.cycles = (double)nk * tile_cost(tile, dtype, c.tiles);
        // from 8 K tiles on (fewer: the adding launch costs more than the serial K loop); slices of at least two K tiles; a lean plan
        // splits up to 64 tiles only, as the smallest-workspace form always did
        if (plan.opts.no_splitk || nk < 8 || c.tiles >= (plan.lean ? 65 : 512)) return c;
        auto cost = [&](int sp) { return (double)((nk + sp - 1) / sp) * tile_cost(tile, dtype, c.tiles * sp) + (c.tiles > 64 ? 6500.0 : 0.0) + 8.0 * sp * M * (double)N / 2200.0; };
        // half-filled grids: K tiles of the fullest CU against 6500 cycles for the adding launch and 2200 bytes per cycle of
        // partial sums (f32 1568 x 256 x 2304: 100 tiles, whole 51 us, five slices 34; 500 x 700 x 1200 37 against 22).  The
        // estimate is good to a sixth: over 700 layers, split where it promised less than that, 89 were slower than whole by
        // more than 3 % (12544 x 6 x 864 in nine slices 36 us against 27), now 17; few channels need a third
        const int most = (int)std::min<int64_t>(std::min<int64_t>(16, c.tiles > 64 ? 16 : 256 / std::max<int64_t>(c.tiles, 1)), nk / 2);
        double best = c.cycles;
        int want = 1;
        for (int sp = 2; sp <= most; ++sp)
            if (cost(sp) < best * 0.95) { best = cost(sp); want = sp; }
        if (c.tiles <= 64) want = most;     // few tiles: as many slices as there are CUs for
        else if (best > c.cycles * (N < 16 ? 0.7 : 0.83)) want = 1;
        if (want < 2 || want * M * N * 4 >= (int64_t)1 << 28) return c;
        c.per = (nk + want - 1) / want;
        c.splits = (nk + c.per - 1) / c.per;
        c.cycles = best;
        return c;
    }

    // Whether a contraction whose channels (features) are no multiple of the 16-byte vector gets zero-padded rows, written by a
    // step of its own, for the vector-load kernels.  The element gather it takes otherwise needs no extra launch and is level
    // at a few K tiles on few workgroups (f32 dense 2 x 90 -> 8: 9 us either way; 10 x 1446 -> 128: 87 us against 16).  From
    // there on the copy, read and written whole at 3 MB per us, must cost less than the K tiles save: us per 64x64 tile and CU,
    // less where the result's rows of channels are stored one element at a time; fitted to 3000 layers of 1 to 467 channels,
    // 1x1 to 7x7, stride 1 and 2, both source and both result layouts (LeNet's one-channel first layer 21 + 7 us padded, 22 as it
    // is; 32 x 467 x 55 x 55 -> 64 1x1 at stride 2 267 against 194).  Of those the K tiles alone would have padded 85 that lose by
    // more than 3 % (up to 1.7x), the copy's cost leaves 7 (up to 1.14x) and gives up 18; it wins 1.7x f32 and 2.0x bf16 on the whole.
    bool pad_k(int x, int wv, int C, int KV, int64_t M, int64_t N, int64_t K, bool concat, int64_t bytes_per_channel, bool slow_store) const
    {
        if (plan.lean || C % KV == 0 || concat || plan.opts.no_dma || g.values[x].role == ROLE_PARAM || consumers[wv].size() != 1) return false;
        const int64_t nk = (K + 8 * KV - 1) / (8 * KV), tiles = ((M + 63) / 64) * ((N + 63) / 64), ld = round_up(C, KV), lim = (int64_t)1 << 30;
        const int64_t nkp = (K / C * ld + 8 * KV - 1) / (8 * KV);
        const double per_tile = KV == 4 ? 2.4 * nk - 0.6 * nkp - (slow_store ? 2.0 : 1.0) : 2.4 * (K / 64 + std::min(1.0, (double)(K % 64) / 8.0)) - 0.3 * nkp + (slow_store ? -1.0 : 0.5);
        const bool pays = (double)bytes_per_channel * (C + ld) / 3e6 < per_tile * (double)std::max<int64_t>(tiles, 256) / 256.0;
        return (nk >= 4 || tiles * nk >= 512) && pays && bytes_per_channel * ld < lim && N * (K / C) * ld * 4 < lim && T(x).dims[0] <= 65535;
    }
    // the weight packing and the contraction's sizes with C filled up to ld
    void pad_gather(PackSpec &pack, IgemmParams &p, const AnchorView *ov, int ld, int KV) const
    {
        const int T_ = p.KH * p.KW;
        pack.gather = 1;
        if (ov) pack.gp = ov->gp;
        else { pack.gp.R = p.N; pack.gp.T = T_; pack.gp.TW = p.KW; pack.gp.s_row = (int64_t)p.C * T_; pack.gp.s_c = T_; pack.gp.s_ti = p.KW; pack.gp.s_tj = 1; }
        pack.gp.dtype = p.in_dtype;
        pack.gp.Cq = ld; pack.gp.Creal = p.C;
        p.C = ld; p.K = p.K1 = ld * T_; p.Kp = (int)round_up(p.K, KV);
    }

    // Whether a contraction runs on the kernel without LDS tiles (igemm_direct.hip), with which tile and K slices (tile 0: no).
    // By two estimates of the call in us, each fitted to 900 conv and dense layers of 1 to 50000 rows (rms 8 to 20 %): launches and
    // latencies, the K steps of the fullest CU, and per workgroup what it starts and ends with.  `other` is the planner's next choice.
    // Taken where it promises a seventh: of drawn layers f32 convolutions that move to 0.58 of the time, bf16 0.52, dense 0.69 and 0.59, LeNet's
    // shape 0.52 and 0.48.  How it is checked: plans with direct_all = 1 against no_direct, layer by layer.
    struct Direct { int tile = 0, slices = 0; };
    enum OtherKind { OTHER_DMA = 0, OTHER_TAPS = 1, OTHER_GATHER = 2 };
    Direct direct_form(int dtype, int64_t M, int64_t N, int64_t K, int mode, int other, bool copies_x, double x_mbytes, bool rides, int taps, bool strided, bool paired, bool pooled, double margin = 0.0, double *estimate = nullptr) const
    {
        Direct best;
        if (plan.opts.no_direct || M * N >= (int64_t)1 << 31) return best;
        const bool bf16 = dtype == RL_BF16;
        const int KV = kv_of(dtype);
        auto cd = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
        // start, per K step alone, per K step of 256 workgroups, per 256 workgroups, and per tile of theirs
        static const double cost32[2][3][5] = {{{5.4, 0.17, 0.40, 0.0, 1.42}, {6.0, 0.13, 0.475, 0.2, 0.86}, {5.0, 0.53, 0.742, 0.37, 0.6}},
                                               {{4.7, 0.31, 0.35, 0.27, 1.03}, {6.0, 0.60, 0.50, 0.39, 0.66}, {4.7, 0.81, 1.2, 0.0, 0.58}}};
        static const double cost16[2][3][4] = {{{3.9, 0.17, 0.42, 1.0}, {5.1, 0.39, 0.40, 1.0}, {4.5, 0.64, 0.59, 0.85}},
                                               {{3.8, 0.18, 0.40, 0.87}, {5.1, 0.73, 0.51, 0.5}, {5.3, 1.0, 1.3, 0.05}}};
        double us = 1e30, us_whole = 1e30, rounds_best = 0.0, steps_best = 0.0;
        for (int form = 0; form < 5; ++form) {
            const int tile = form < 4 ? 32 : 16, slices = form < 4 ? 1 << form : 8, wt = 8 / slices;
            if (plan.opts.no_splitk && slices > 1) continue;
            if (plan.opts.direct_all > 1 && (tile != plan.opts.direct_all / 16 || slices != plan.opts.direct_all % 16)) continue;
            const double steps = (double)cd(cd(K, KV * (64 / tile)), slices), rounds = (double)(cd(M, tile * wt) * cd(N, tile)) / 256.0;
            const double *c = tile == 32 ? cost32[bf16][mode] : cost16[bf16][mode];
            // the chunk's tap; at a stride a tap's pixels fill half of their cache lines, and the next tap comes back for the rest too late
            const double per = c[2] + (mode == DIRECT_ROWS && taps > 1 ? 0.1 : 0.0), lines = strided && mode != DIRECT_ROWS ? 1.0 + 0.02 * taps : 1.0;
            auto at = [&](double r) { return c[0] + lines * std::max(c[1] * steps, per * steps * std::max(r, 1.0)) + (c[3] + (tile == 32 ? c[4] * wt : 0.0)) * rounds; };
            if (at(rounds) < us) { us = at(rounds); us_whole = at(std::ceil(rounds)); best.tile = tile; best.slices = slices; rounds_best = rounds; steps_best = steps; }
        }
        if (estimate) *estimate = us;
        if (plan.opts.direct_all || estimate) return best;      // the caller compares
        // A last round that only some of the CUs have a workgroup for.  Rows of f32 features read one by one: it counts in full, as two
        // workgroups on a CU have twice the lines in use that the vector L1 holds (354 x 704 x 1066 19.2 us by padded rows, 33.2 so; 249 x 1172 x
        // 1013 19.0 and 37.3); shorter rows still fit (1118 x 364 x 326 17.6 and 12.5).  Taps of channels in planes, a last round less than half full:
        // it counts by half, from so many K steps a slice that the other kernels' longer start is made up for, earlier at a stride, where the lines
        // fetched are half used (32x304x37x37 -> 78 3x3 at stride 2 41 and 53).  Not up to 32 channels, where the other kernels' estimate, of tiles
        // that are half empty, is low itself, nor where a max-pool of the result rides along.  It takes 195 of 90000 drawn layers off
        // this kernel, which then run in 0.84 of the time; 15 of them lose more than 3 %, up to 1.15x.
        if (rounds_best > 1.0 && !pooled) {
            if (!bf16 && mode == DIRECT_ANY && taps == 1 && other == OTHER_DMA && steps_best >= 10 && N > 128) us = us_whole;
            else if (mode == DIRECT_PLANES && taps > 1 && steps_best >= (strided ? 16 : 32) && N > 32 && rounds_best - std::floor(rounds_best) < 0.5) us = 0.5 * (us + us_whole);
        }
        const KSlices lds = k_slices(direct_load_tile(dtype, M, N), dtype, M, N, K);
        const bool split = lds.splits > 1;
        static const double otherc[2][3][6] = {{{4.5, 1.04, 3.2, 2.8, 0.48, 0.63}, {5.0, 1.15, 3.5, 2.8, 0.35, 0.69}, {11.0, 2.3, 3.0, 0.0, 0.0, 1.09}},
                                               {{3.9, 0.95, 4.3, 3.7, 0.95, 1.64}, {6.1, 1.11, 3.1, 2.1, 0.67, 1.52}, {15.5, 4.4, 5.0, 0.0, 0.0, 0.84}}};
        const double *c = otherc[bf16][other];
        const double theirs = c[0] + c[1] * lds.cycles / 2100.0 + (split ? c[2] : 0.0) + (copies_x ? c[3] + c[4] * x_mbytes : 0.0) +
                              c[5] * M * (double)N * dtype_size(dtype) / 1e6 - (rides && split ? 3.0 : 0.0) - (paired ? 3.5 : 0.0);
        // (few slices: short K on many tiles, where the stores decide and the estimates are at their worst)
        return us < (margin > 0.0 ? margin : best.slices < 4 && other != OTHER_GATHER ? 0.7 : 0.85) * theirs ? best : Direct();
    }

    // The same where the pixel-on-lane kernels would run, on 64x64 tiles: layers of a channel-last network at small batches.  They
    // take 3.05 us and 0.244 a K tile, once more for every 256 tiles; this kernel 0.67 of the estimate above there, dense layers 0.8 (91 drawn convolutions of 64 to 512
    // channels, rms 9 and 15 %).  Taken where it promises a seventh: 36 of them move, to 0.70 of their time, none loses
    // (2x128x7x7 -> 128 3x3 6.6 -> 3.8 us; 4x192x14x14 10.7 -> 7.6; the residual network's shape, one image, 158 -> 124).
    Direct direct_before_lp(int64_t M, int64_t N, int64_t K, int taps, bool strided, double of_estimate) const
    {
        auto cd = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
        if (cd(M, 128) * cd(N, 64) >= 192) return Direct();
        double us = 0.0;
        const Direct best = direct_form(RL_BF16, M, N, K, DIRECT_ROWS, OTHER_DMA, false, 0.0, false, taps, strided, false, false, 0.0, &us);
        const double theirs = 3.05 + 0.244 * (double)cd(K, 64) * std::max(1.0, (double)(cd(M, 64) * cd(N, 64)) / 256.0);
        return us > 0.0 && of_estimate * us < 0.85 * theirs ? best : Direct();
    }

    static bool pool_2x2(const OpNode &o)
    {
        const auto &a = o.attrs;
        return o.kind == RL_OP_MAXPOOL2D && a.kernel[0] == 2 && a.kernel[1] == 2 && a.stride[0] == 2 && a.stride[1] == 2 && a.pad[0] == 0 && a.pad[1] == 0;
    }

    // the gradient with respect to the input may go out with the one with respect to the weights (pair_gradients)
    bool beside_weights_gradient(int dy) const
    {
        if (plan.opts.no_pair || plan.lean) return false;
        for (int c : consumers[dy])
            if ((g.ops[c].kind == RL_OP_DENSE_GRAD_W || g.ops[c].kind == RL_OP_CONV2D_GRAD_W) && g.ops[c].in[0] == dy && tn_ok(g.ops[c])) return true;
        return false;
    }

    rl_status plan_anchor(int gi, const std::vector<int> &ops, const AnchorView *ov = nullptr)
    {
        std::set<int> gset(ops.begin(), ops.end());
        size_t ai = 0;
        int x = -1, x2 = -1;
        if (g.ops[ops[0]].kind == RL_OP_CONCAT) {
            ai = 1;
            const OpNode &cc = g.ops[ops[0]];
            if (g.ops[ops[1]].in[0] != cc.out[0]) return fail(RL_ERR_UNSUPPORTED, "concat must feed the dense's first operand");
            x = cc.in[0];
            x2 = cc.in[1];
        }
        const OpNode &an = g.ops[ops[ai]];
        const int akind = ov ? ov->kind : an.kind;
        if (x < 0) x = an.in[0];
        const int wv = an.in[1];
        if (g.values[wv].role != ROLE_PARAM) return fail(RL_ERR_UNSUPPORTED, "contraction weights must be a param");
        const int in_dt = T(x).dtype;
        const int KV = kv_of(in_dt);
        const bool gates = g.ops[ops.back()].kind == RL_OP_LSTM_GATES && ops.size() > ai + 1;
        Chain chain;
        rl_status st = build_chain(ops, ai + 1, gates ? ops.size() - 1 : ops.size(), an.out[0], gset, chain);
        if (st != RL_OK) return st;
        if (chain.bias_axis >= 0 && chain.bias_axis != 1) return fail(RL_ERR_UNSUPPORTED, "bias_add fused into a contraction must be along axis 1");
        if (gates) {
            const OpNode &go = g.ops[ops.back()];
            const int cprod = g.values[go.in[1]].producer;
            if (go.in[0] != chain.last_value || (cprod >= 0 && gset.count(cprod))) return fail(RL_ERR_UNSUPPORTED, "fused group is not a single chain");
        }
        if (gates)
            for (int i = 0; i < chain.epi.n_ops; ++i)
                if (epi_host_op(chain.epi, i) != E_BIAS) return fail(RL_ERR_UNSUPPORTED, "only bias_add may sit between the contraction and lstm_gates");

        IgemmParams p{};
        IgemmLaunch il{};
        PackSpec pack;
        bool need_pack = false, padded = false;       // padded: contraction channels (features) filled up with zeros to whole vectors
        int xbuf = -1, x2buf = -1;
        double flops = 0.0;
        size_t x_extent = 0;                 // bytes of the tensor the kernel reads as x
        const rl_type &ot = T(an.out[0]);
        p.in_dtype = in_dt;
        int out_layout = L_NATIVE;
        const int vout = gates ? -1 : chain.last_value;

        // form of the injective chain, needed before the kernel variant is chosen
        Epilogue cls = chain.epi;
        finalize_epilogue(cls);
        const bool epi_any = cls.simple && (!cls.has_bias || cls.bias_dtype == DT_F32) && (cls.t_op < 0 || (cls.t_op == E_ADD && cls.t_dtype == DT_BF16));
        const bool relu_form = cls.rest_n == 0 || cls.relu_last;     // at most one ReLU behind them: every pixel-on-lane kernel; anything else: the general one
        const bool epi_lp = epi_any && relu_form;
        bool stem = false;
        Direct direct;
        int direct_mode = 0;
        const size_t lim = (size_t)1 << 31;

        if (akind == RL_OP_CONV2D) {
            const rl_type &xt = T(x), &wt = T(wv);
            p.C = (int)xt.dims[1]; p.H = (int)xt.dims[2]; p.W = (int)xt.dims[3];
            const bool xov = ov && ov->xbuf >= 0;
            if (xov) { p.H = ov->xH; p.W = ov->xW; if (ov->xC) p.C = ov->xC; }
            const size_t x_own = xov ? (size_t)xt.dims[0] * p.H * p.W * p.C * dtype_size(in_dt) : bytes_of(x);
            p.KH = (int)wt.dims[2]; p.KW = (int)wt.dims[3];
            p.OH = (int)ot.dims[2]; p.OW = (int)ot.dims[3]; p.OHW = p.OH * p.OW;
            p.sh = an.attrs.stride[0]; p.sw = an.attrs.stride[1]; p.ph = an.attrs.pad[0]; p.pw = an.attrs.pad[1];
            p.N = (int)wt.dims[0];
            if (ov) { p.N = ov->N; p.KH = ov->KH; p.KW = ov->KW; p.sh = p.sw = 1; p.ph = ov->ph; p.pw = ov->pw; }
            if (xt.dims[0] * (int64_t)p.OHW > 0x7fffffff) return fail(RL_ERR_UNSUPPORTED, "conv2d too large");
            p.M = (int)(xt.dims[0] * p.OHW); p.K = p.C * p.KH * p.KW; p.K1 = p.K;
            p.Kp = (int)round_up(p.K, KV);
            out_layout = (vout >= 0 && out_set.count(vout)) ? L_NATIVE : L_NHWC;
            flops = 2.0 * p.M * (double)p.N * p.K;
            const int64_t bytes_per_channel = xt.dims[0] * (int64_t)p.H * p.W * dtype_size(in_dt);
            const bool pad = !xov && pad_k(x, wv, p.C, KV, p.M, p.N, p.K, x2 >= 0, bytes_per_channel, out_layout == L_NHWC && p.N % 8 != 0);
            if (vout >= 0 && x2 < 0 && !gates && x_own < lim && (size_t)p.N * p.Kp * dtype_size(in_dt) < lim) {
                const bool last = xov || phys[L_NHWC][x] >= 0, vec = p.C % KV == 0;
                direct_mode = !vec ? DIRECT_ANY : last ? DIRECT_ROWS : DIRECT_PLANES;
                const int next = !out_set.count(vout) && consumers[vout].size() == 1 ? consumers[vout][0] : -1;
                const bool pooled = next >= 0 && cls.simple && cls.t_op < 0 && pool_2x2(g.ops[next]);       // fuse_direct_store
                // bf16 channels in whole K tiles: against the pixel-on-lane kernels where those would run (from channels in planes, which they
                // get copied, never)
                const bool lp_next = in_dt == RL_BF16 && p.C % 64 == 0 && p.N % 8 == 0 && p.KH * p.KW <= 32 && epi_any && T(vout).dtype == RL_BF16 && !plan.opts.no_lp &&
                                     (out_layout == L_NHWC || (flops >= 4e8 && !plan.opts.no_out_transpose));
                // 3x3 from 64 to 64 channels has a kernel and a packing of its own (conv3x3_c64.hip) and keeps them from planes too
                const bool c64 = in_dt == RL_BF16 && p.C == 64 && p.N == 64 && p.KH == 3 && p.KW == 3 && !ov && !last;
                // a strided convolution and the projection of the same input go out together (pair_contractions)
                int strided = 0;
                for (int c : consumers[x]) strided += g.ops[c].kind == RL_OP_CONV2D && g.ops[c].attrs.stride[0] > 1;
                if (c64 && !plan.opts.direct_all) {}
                else if (lp_next && !plan.opts.direct_all) {
                    if (last && strided < 2 && !ov) direct = direct_before_lp(p.M, p.N, p.K, p.KH * p.KW, p.sw > 1, 0.67);
                } else
                    direct = direct_form(in_dt, p.M, p.N, p.K, direct_mode, !vec && !pad ? OTHER_GATHER : p.C % (8 * KV) == 0 ? OTHER_DMA : OTHER_TAPS,
                                         (!last || pad) && consumers[x].size() == 1, (double)x_own / 1e6, false, p.KH * p.KW, p.sw > 1, ov && beside_weights_gradient(x), pooled);
            }
            // A bf16 result that is a graph output (Shape order): the slower direct-load kernel stores in that order
            // itself, the pixel-on-lane kernels only where fuse_planes_store lets them.  From 0.4 GFLOP on, the pixel-on-lane kernels writing channel-last into the workspace plus a
            // transposition (one launch more, and one more for a channel-first residual) are faster: 64x128x28x28 through
            // 3x3 20 + 9 us against 56, with a residual 43 against 166; at 0.46 GFLOP 14.3 against 16.9; below, the
            // direct-load kernel with its K split is level or ahead (0.23 GFLOP: 16.4 against 14.6).
            if (out_layout == L_NATIVE && vout >= 0 && !plan.opts.no_out_transpose && !plan.opts.no_lp && in_dt == RL_BF16 && T(vout).dtype == RL_BF16 &&
                p.C % 64 == 0 && p.N % 8 == 0 && p.KH * p.KW <= 32 && x2 < 0 && !gates && epi_any && flops >= 4e8 &&
                channel_last_output_of(vout) < 0)
                out_layout = L_NHWC;
            if (out_layout == L_NHWC) { p.ys_n = (int64_t)p.OHW * p.N; p.ys_p = p.N; p.ys_c = 1; }
            else { p.ys_n = (int64_t)p.N * p.OHW; p.ys_p = 1; p.ys_c = p.OHW; }
            // Few-channel stem (e.g. 3 -> 64, 7x7, stride 2): gathering single elements starves the MFMAs.  Copy the
            // input into a zero-padded 4-channel channel-last frame instead; a K tile then holds two filter rows of
            // 8 pixels x 4 channels and travels by direct loads like any other (see launch_stem_pad).
            const int KH2 = (p.KH + 1) / 2;
            const int64_t Hp = (int64_t)(p.OH - 1) * p.sh + 2 * KH2, Wp = (int64_t)(p.OW - 1) * p.sw + 8;
            const size_t frame = (size_t)xt.dims[0] * Hp * Wp * 8;
            stem = in_dt == RL_BF16 && p.C <= 4 && p.KW <= 8 && p.sw % 2 == 0 && KH2 <= 32 && epi_lp && vout >= 0 && T(vout).dtype == RL_BF16 &&
                   out_layout == L_NHWC && p.N % 8 == 0 && bytes_of(vout) < lim && frame < lim && phys[L_NATIVE][x] >= 0 && !plan.opts.no_stem && !ov;
            if (stem) {
                direct = Direct();
                int xnat;
                st = need(x, L_NATIVE, xnat);
                if (st != RL_OK) return st;
                xbuf = new_ws(frame);
                Step &ps = add_step(S_STEM_PAD, "stem_pad", "stem_pad_nhwc4");
                ps.t_N = (int)xt.dims[0]; ps.t_C = p.C; ps.st_H = p.H; ps.st_W = p.W; ps.st_Hp = (int)Hp; ps.st_Wp = (int)Wp;
                ps.st_ph = p.ph; ps.st_pw = p.pw;
                ps.slot[SL_X] = xnat; ps.slot[SL_Y] = xbuf;
                ps.bytes = (double)bytes_of(x) + (double)frame;
                pack.dtype = in_dt; pack.O = p.N; pack.C = p.C; pack.KH = p.KH; pack.KW = p.KW; pack.stem = 1; pack.T = p.KH * p.KW;
                // the contraction as the kernel sees it: 64 "channels" per tap, KH2 taps, taps two frame rows apart
                p.C = 64; p.KH = KH2; p.KW = 1; p.H = (int)Hp; p.W = (int)Wp; p.ph = 0; p.pw = 0;
                p.xs_n = Hp * Wp * 4; p.xs_h = Wp * 4; p.xs_w = 4; p.xs_c = 1;
                p.ts_h = 2 * Wp * 4; p.ts_w = 0; p.seg_stride = (uint32_t)(Wp * 8);
                p.K = KH2 * 64; p.K1 = p.K; p.Kp = p.K;
                pack.Kp = p.Kp; pack.perm_block = 0;
                il.avec = 1;
                need_pack = true;
                x_extent = frame;
            } else if (pad && !direct.tile) {
                // a channel count that is no multiple of the vector: rows padded with zeros, weights likewise
                int ld;
                plan.spent = true;
                st = need_rows(gi, x, xbuf, ld);
                if (st != RL_OK) return st;
                pad_gather(pack, p, ov, ld, KV);
                p.xs_n = (int64_t)p.H * p.W * ld; p.xs_h = (int64_t)p.W * ld; p.xs_w = ld; p.xs_c = 1;
                p.ts_h = p.xs_h; p.ts_w = p.xs_w; p.seg_stride = 64;
                il.avec = 1;
                need_pack = padded = true;
                pack.dtype = in_dt; pack.O = p.N; pack.C = p.C; pack.T = p.KH * p.KW; pack.Kp = p.Kp; pack.perm_block = -3;
                x_extent = (size_t)xt.dims[0] * p.H * p.W * ld * dtype_size(in_dt);
            } else {
                il.avec = (p.C % KV == 0);
                int xl;
                if (direct.tile) xl = xov || phys[L_NHWC][x] >= 0 ? L_NHWC : L_NATIVE;
                else if (il.avec || xov) xl = L_NHWC;
                else xl = phys[L_NATIVE][x] >= 0 ? L_NATIVE : L_NHWC;
                if (xov) xbuf = ov->xbuf;
                else st = need(x, xl, xbuf);
                if (st != RL_OK) return st;
                if (xl == L_NHWC) { p.xs_n = (int64_t)p.H * p.W * p.C; p.xs_h = (int64_t)p.W * p.C; p.xs_w = p.C; p.xs_c = 1; }
                else { p.xs_n = (int64_t)p.C * p.H * p.W; p.xs_c = (int64_t)p.H * p.W; p.xs_h = p.W; p.xs_w = 1; }
                p.ts_h = p.xs_h; p.ts_w = p.xs_w; p.seg_stride = 64;
                need_pack = !(p.KH * p.KW == 1 && p.C % KV == 0) || ov;
                pack.dtype = in_dt; pack.O = p.N; pack.C = p.C; pack.T = p.KH * p.KW; pack.Kp = p.Kp; pack.perm_block = 0;
                x_extent = x_own;
            }
        } else {
            const rl_type &wt = T(wv);
            const int64_t K = ov ? T(x).dims[1] : wt.dims[1], Nf = ov ? ov->N : wt.dims[0];
            if (ot.dims[0] > 0x7fffffff || K > 0x7ffffff0 || Nf > 0x7fffffff) return fail(RL_ERR_UNSUPPORTED, "dense too large");
            p.M = (int)ot.dims[0]; p.N = (int)Nf; p.K = (int)K; p.Kp = (int)round_up(K, KV);
            p.C = p.K; p.H = p.W = p.KH = p.KW = p.OH = p.OW = p.OHW = 1; p.sh = p.sw = 1;
            p.K1 = x2 >= 0 ? (int)T(x).dims[1] : p.K;
            const int K2 = p.K - p.K1;
            il.avec = (p.K1 % KV == 0) && (K2 % KV == 0);
            // a layer of at most 64 outputs behind another layer keeps its own rows: it may ride on that layer's adding launch
            const bool may_chain = p.N <= REDUCE_DENSE_MAX_N2 && g.values[x].producer >= 0;
            const bool pad = !il.avec && !gates && !may_chain && pad_k(x, wv, p.K, KV, p.M, p.N, p.K, x2 >= 0, (int64_t)p.M * dtype_size(in_dt), false);
            if (vout >= 0 && x2 < 0 && !gates && bytes_of(x) < lim && (size_t)p.N * round_up(p.K, 8 * KV) * dtype_size(in_dt) < lim) {
                // a split layer whose adding launch also runs the small layer behind it (chain_small_dense) is one launch for two already
                const int next = !out_set.count(vout) && consumers[vout].size() == 1 ? consumers[vout][0] : -1;
                const bool rides = next >= 0 && p.N <= REDUCE_DENSE_MAX_N1 && g.ops[next].kind == RL_OP_DENSE && T(g.ops[next].out[0]).dims[1] <= REDUCE_DENSE_MAX_N2 &&
                                   !plan.opts.no_splitk;
                const int64_t nk = (K + 8 * KV - 1) / (8 * KV);
                direct_mode = il.avec ? DIRECT_ROWS : DIRECT_ANY;
                // with more than 256 tiles of 32 x 32 the kernels with LDS tiles are level or ahead.  With few K tiles, or bf16 K in whole ones, this
                // kernel is ahead wherever its estimate is below theirs: of 124 drawn layers that went to LDS tiles before, 66 move, bf16 to 0.67
                // of their time (28 x 446 x 320 8.2 -> 3.8 us, 48 x 980 x 1280 9.8 -> 5.4), f32 to 0.58, none loses; before the pixel-on-lane kernels
                // (bf16, K in whole tiles, N in eights) 38 of 97 to 0.75, one loses 3 % (16 x 64 x 1024 6.1 -> 4.7)
                // (not the gradients, which may go out in pairs, nor a layer that may ride on the adding launch of the one before)
                const bool short_k = il.avec && (nk <= (in_dt == RL_F32 ? 4 : 8) || (in_dt == RL_BF16 && p.K % 64 == 0));
                bool behind_split = false;
                for (const Step &f : plan.steps) behind_split |= f.kind == S_IGEMM && f.slot[SL_Y] >= 0 && f.slot[SL_Y] == phys[L_NATIVE][x] && f.il.splits > 1;
                const bool many = il.avec && (rides || (short_k && behind_split) || ((ot.dims[0] + 31) / 32) * ((Nf + 31) / 32) > 256), lds = many || (il.avec && short_k && ov);
                const bool lp_next = in_dt == RL_BF16 && p.K % 64 == 0 && p.N % 8 == 0 && epi_any && T(vout).dtype == RL_BF16 && !plan.opts.no_lp;
                if (lp_next && !plan.opts.direct_all) {
                    if (!many && relu_form) direct = direct_before_lp(p.M, p.N, p.K, 1, false, 0.8);
                } else if (plan.opts.direct_all || !lds)
                    direct = direct_form(in_dt, p.M, p.N, p.K, direct_mode, il.avec || pad ? OTHER_DMA : OTHER_GATHER, pad && consumers[x].size() == 1, (double)bytes_of(x) / 1e6, rides, 1, false, ov && beside_weights_gradient(x), false,
                                         short_k ? 0.95 : 0.0);
            }
            if (pad && !direct.tile) {
                int ld;
                plan.spent = true;
                flops = 2.0 * p.M * (double)p.N * p.K;
                st = need_rows(gi, x, xbuf, ld);
                if (st != RL_OK) return st;
                pad_gather(pack, p, ov, ld, KV);
                il.avec = 1;
                padded = true;
            } else st = need(x, L_NATIVE, xbuf);
            if (st != RL_OK) return st;
            if (x2 >= 0) { st = need(x2, L_NATIVE, x2buf); if (st != RL_OK) return st; }
            p.xs_n = p.K1; p.xs_c = 1; p.xs_h = 0; p.xs_w = 0; p.x2s_n = K2;
            p.ts_h = 0; p.ts_w = 0; p.seg_stride = 64;
            if (!padded) flops = 2.0 * p.M * (double)p.N * p.K;
            x_extent = padded ? (size_t)p.M * p.K * dtype_size(in_dt) : bytes_of(x);
            need_pack = (p.K % KV != 0) || gates || ov || padded;
            pack.dtype = in_dt; pack.O = p.N; pack.C = p.K; pack.T = 1; pack.Kp = p.Kp; pack.perm_block = padded ? -3 : gates ? 64 : 0;
            p.ys_n = p.N; p.ys_p = p.N; p.ys_c = 1;
        }
        // 3x3 bf16 weights from 64 to 64 channels carry, behind the matrix, a second copy in the fragment order of the
        // kernel that keeps them in registers (whichever kernel a step ends up with, so that every user agrees)
        const bool dual = !ov && akind == RL_OP_CONV2D && !stem && in_dt == RL_BF16 && p.N == 64 && p.C == 64 && p.KH == 3 && p.KW == 3 && p.Kp == p.K;
        if (dual) pack.perm_block = -1;
        pack.bytes = (size_t)pack.O * pack.Kp * dtype_size(in_dt);
        // a convolution's weights for the kernel without LDS tiles, used by it alone: packed in the order of its fragments (where they
        // are packed in any case: which params are is the same in every form of a plan).  Not of a single pixel through one tap, which is a
        // dense layer and may ride on the adding launch of the one before it (chain_small_dense), whose kernel reads rows
        p.w_frag = akind == RL_OP_CONV2D && !ov && direct.tile && need_pack && pack.perm_block == 0 && !dual && consumers[wv].size() == 1 && (p.OHW > 1 || p.KH * p.KW > 1) ? 1 : 0;
        const int64_t frag_k = round_up(p.K, KV * (64 / std::max(direct.tile, 1)));
        const size_t frag_bytes = (size_t)round_up(pack.O, std::max(direct.tile, 1)) * frag_k * dtype_size(in_dt);
        if (p.w_frag && frag_bytes < lim) {
            pack.perm_block = -direct.tile;
            p.Kp = pack.Kp = (int)frag_k;
            pack.bytes = frag_bytes;
        } else p.w_frag = 0;                 // filled up to whole tiles they would pass what the kernel's offsets reach
        // the vector-load kernel addresses its operands with 32-bit byte offsets and wants a K tile
        // (128 bytes per row) to lie inside one operand of a concatenation
        {
            if (x_extent >= lim || pack.bytes >= lim || (x2 >= 0 && bytes_of(x2) >= lim)) il.avec = 0;
            if (x2 >= 0 && p.K1 % (8 * KV) != 0) il.avec = 0;
            p.x_bytes = (uint32_t)std::min(x_extent, lim - 1);
            p.x2_bytes = x2 >= 0 ? (uint32_t)std::min(bytes_of(x2), lim - 1) : 0;
            p.w_bytes = (uint32_t)std::min(pack.bytes, lim - 1);
            if (dual) pack.bytes *= 2;
            // LDS-DMA variant: a K tile must lie inside one filter tap (and one concat operand)
            const int bke = 8 * KV;
            const size_t halo = (size_t)((int64_t)p.ph * p.xs_h + (int64_t)p.pw * p.xs_w) * dtype_size(in_dt);
            il.dma = !stem && il.avec && p.C % bke == 0 && p.K % bke == 0 && p.K / bke >= 2 && p.KH * p.KW <= 32 &&
                     (x2 < 0 || p.K1 % bke == 0) && x_extent + halo < lim && !plan.opts.no_dma;
            // a dense contraction whose K is a multiple of the vector but not of the K tile: the weights are packed
            // with zeros up to whole tiles and the kernel requests the activation chunks past K out of range
            if (!il.dma && akind == RL_OP_DENSE && !stem && !gates && x2 < 0 && il.avec && p.K % bke != 0 && p.K / bke >= 2 &&
                x_extent < lim && (size_t)p.N * round_up(p.K, bke) * dtype_size(in_dt) < lim && !plan.opts.no_dma) {
                il.dma = 1;
                p.Kp = (int)round_up(p.K, bke);
                need_pack = true;
                pack.Kp = p.Kp;
                pack.bytes = (size_t)pack.O * pack.Kp * dtype_size(in_dt);
                p.w_bytes = (uint32_t)pack.bytes;
            }
            // pixel-on-lane variant: bf16 throughout, output rows contiguous in n, epilogue [bias] [+residual] [relu]
            bool y_ok = vout >= 0 && T(vout).dtype == RL_BF16 && p.ys_c == 1 && p.ys_n == (int64_t)p.OHW * p.ys_p && p.N % 8 == 0 &&
                        bytes_of(vout) < lim;
            il.lp = stem || (il.avec && in_dt == RL_BF16 && p.C % bke == 0 && p.K % bke == 0 && p.KH * p.KW <= 32 && x2 < 0 && !gates &&
                             x_extent + halo < lim && epi_any && y_ok && !plan.opts.no_lp);
            // A very long K on few tiles (late layers at small batches): the pixel-on-lane kernels do not cut K, the direct-load
            // kernel does.  From 64 K tiles on, on 2 to 64 tiles of 64x64, that is worth its adding launch (98 x 512 x 4608: 24 us
            // against 15.5; 36 K tiles are level, 15 us either way).
            const int64_t lp_tiles = (int64_t)((p.M + 63) / 64) * ((p.N + 63) / 64);
            if (il.lp && !stem && il.dma && p.K / bke >= 64 && lp_tiles >= 2 && lp_tiles <= 64 && !plan.opts.no_splitk && !plan.lean) il.lp = 0;
            // everything else whose chunks are whole: K tiles that span taps (or a dense of less than two).  Not for bf16 results in whole
            // rows of channels on 300 tiles of 128x128 and more: the register-staged kernel runs two such workgroups per CU (64x200x28x28
            // -> 128 3x3: 74 us against 83, 128 such layers 1.05 on average; fewer tiles or channel-first results 0.72 to 0.94)
            const bool many_rows = in_dt == RL_BF16 && p.ys_c == 1 && p.N > 64 && p.N % 8 == 0 && (int64_t)((p.M + 127) / 128) * ((p.N + 127) / 128) >= 300;
            if (!il.dma && !il.lp && il.avec && !stem && !gates && x2 < 0 && !many_rows && x_extent + halo < lim && pack.bytes < lim && !plan.opts.no_dma) {
                il.dma = il.taps = 1;
                make_fast_div((uint32_t)p.C, p.div_c_mul, p.div_c_sh);
                make_fast_div((uint32_t)p.KW, p.div_kw_mul, p.div_kw_sh);
            }
            il.anyact = il.lp && !stem && !relu_form;
            // weights-stationary persistent variant: pays off when the weights leave LDS for a deep ring (K <= 320);
            // the plan option ws_all also takes it up to K = 576, where its shallower ring is latency-bound
            il.ws = il.lp && !il.anyact && p.N <= 64 && (p.K / bke <= 5 || (p.K / bke <= 9 && plan.opts.ws_all)) && !plan.opts.no_ws;
            // 3x3 / stride 1 / pad 1 from 64 to 64 channels on rows of at most 63 pixels: weights in registers, every
            // input pixel fetched once per region
            il.c64 = il.lp && !il.anyact && !stem && akind == RL_OP_CONV2D && p.C == 64 && p.N == 64 && p.KH == 3 && p.KW == 3 && p.sh == 1 && p.sw == 1 &&
                     p.ph == 1 && p.pw == 1 && p.OH == p.H && p.OW == p.W && p.W <= 63 && p.Kp == p.K && p.ys_p == 64 && !plan.opts.no_c64;
            il.c64 = il.c64 && dual;
            if (il.c64) { il.ws = 0; p.w_bytes = (uint32_t)pack.bytes; }
            p.y_bytes = vout >= 0 ? (uint32_t)std::min(bytes_of(vout), lim - 1) : 0;
            make_fast_div((uint32_t)p.OHW, p.div_ohw_mul, p.div_ohw_sh);
            make_fast_div((uint32_t)p.OW, p.div_ow_mul, p.div_ow_sh);
            p.tap_rep = 0;
            if (p.KH * p.KW <= 32)
                for (int kh = 0; kh < p.KH; ++kh) p.tap_rep |= 1u << (kh * p.KW);
        }
        if (ov && !padded) { pack.gather = 1; pack.gp = ov->gp; pack.perm_block = -3; }
        if (pack.gather) pack.gp.Kp = pack.Kp;
        if (need_pack) {
            auto it = plan.packs.find(wv);
            if (it != plan.packs.end() && (ov || it->second.perm_block != pack.perm_block || it->second.Kp != pack.Kp))
                return fail(RL_ERR_UNSUPPORTED, "one param needs two different kernel-native layouts");
            plan.packs[wv] = pack;
        } else if (plan.packs.count(wv)) {
            return fail(RL_ERR_UNSUPPORTED, "one param needs two different kernel-native layouts");
        }

        // (whether and how the weights are packed does not depend on this choice)
        if (direct.tile) {
            il = IgemmLaunch{};
            il.direct = 1 + direct_mode;
            il.direct_tile = direct.tile; il.direct_slices = direct.slices;
            make_fast_div((uint32_t)p.C, p.div_c_mul, p.div_c_sh);
            make_fast_div((uint32_t)p.KW, p.div_kw_mul, p.div_kw_sh);
        }

        // tile: the largest that still yields enough workgroups for 256 CUs
        auto nblk = [&](int bm, int bn) { return (int64_t)((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn); };
        if (gates) {
            il.tile = TILE_64x64;
            il.gates = 1;
            int64_t Hd = T(g.ops[ops.back()].in[1]).dims[1];
            if (Hd % 16 != 0) return fail(RL_ERR_UNSUPPORTED, "fused gate epilogue needs hidden size divisible by 16");
            p.hidden = (int)Hd;
            p.h_dtype = T(g.ops[ops.back()].out[1]).dtype;
            const int64_t K2 = p.K - p.K1;
            // the step without LDS tiles (igemm_direct.hip), except for bf16 cells that rl_plan_run_recurrent may hoist, and where the
            // direct-load kernel is ahead, which fetches its fragments once per 64 rows (2048 x 256 units from 256, f32: 27 us against 52; 512:
            // 17.3 against 16.2; bf16 9.6 and 10.3).  Estimates in us: 50 cycles a load on either side of 16 rows and 4 units, a K tile per tile_cost.
            const int64_t rows16 = ((int64_t)p.M + 15) / 16;
            const int units = rows16 * (Hd / 16) < 64 ? 4 : 8;       // measured 4 / 8 / 16 at 32 to 63 blocks of 16 x 16: 0.18 / 0.22 / 0.33 of the gather's time, at 64 to 127 0.32 / 0.28 / 0.42
            const double direct_us = 3.6 + (double)(rows16 * Hd / 8) / 256.0 * (double)(p.K / (4 * KV)) * 200.0 / 2100.0;
            const double dma_us = 5.5 + (double)(p.K / (8 * KV)) * tile_cost(TILE_64x64, in_dt, (p.M + 63) / 64 * (Hd / 16)) / 2100.0;
            const bool keep = il.dma && (in_dt == RL_BF16 ? p.K1 >= 128 || dma_us < direct_us : dma_us < direct_us);
            if (x2 >= 0 && p.K1 % KV == 0 && K2 % KV == 0 && x_extent < lim && bytes_of(x2) < lim && pack.bytes < lim && chain.epi.n_ops <= 1 && p.M <= 65535 * 16 && !plan.opts.no_direct &&
                (!keep || plan.opts.direct_all)) {
                il = IgemmLaunch{};
                il.tile = TILE_64x64;
                il.gates = il.direct = 1;
                il.direct_tile = 16; il.direct_slices = 8;
                il.direct_units = plan.opts.direct_all > 1 ? (plan.opts.direct_all % 16 == 4 ? 4 : 8) : units;
                p.w_bytes = (uint32_t)pack.bytes;
            }
        } else if (!il.avec) {
            il.tile = TILE_64x64;
        } else if (il.taps || (il.dma && in_dt == RL_F32)) {
            il.tile = direct_load_tile(in_dt, p.M, p.N);
        } else if (il.lp && p.N > 64 && nblk(256, 128) >= 190 && !plan.opts.no_lp_256) {
            il.tile = TILE_256x128;        // a quarter fewer operand bytes per MFMA than 128x128
        } else if (p.N > 64 && nblk(128, 128) >= 192) {
            il.tile = TILE_128x128;
        } else if (nblk(128, 64) >= 192) {
            il.tile = TILE_128x64;
        } else {
            il.tile = TILE_64x64;
        }

        // a dense, or a 1x1 convolution at stride 1, large enough for 256x256 tiles
        il.big = il.lp && !il.anyact && !il.ws && !stem && il.tile == TILE_256x128 && p.KH * p.KW == 1 && p.sh == 1 && p.sw == 1 && p.ph == 0 && p.pw == 0 &&
                 igemm_big_better(p.M, p.N, p.K);

        // 3x3 / stride 1 / pad 1 on short image rows with whole 64-channel slices: the nine taps of a slice are read
        // from one copy of the input rows (needs one of the larger tiles)
        il.run = il.lp && !il.anyact && !il.c64 && !il.ws && !stem && akind == RL_OP_CONV2D && p.KH == 3 && p.KW == 3 && p.sh == 1 && p.sw == 1 && p.ph == 1 &&
                 p.pw == 1 && p.OH == p.H && p.OW == p.W && p.W <= 30 && p.C % 64 == 0 && p.Kp == p.K && il.tile != TILE_64x64 &&
                 !plan.opts.no_run;
        if (il.run && il.tile == TILE_128x64 && p.C % 128 == 0 && !plan.opts.no_run_ks) {
            il.run = 2;                                                 // K split over the waves
            // weights of all channel tiles larger than an XCD's share of L2 (4 MB): tiles are numbered channel-tile-major,
            // so that an XCD multiplies every pixel tile by one channel tile's weights
            p.nmajor = (int64_t)p.N * p.K * 2 > (3 << 20) ? 1 : 0;
        }

        double bytes = (double)bytes_of(x) + (x2 >= 0 ? (double)bytes_of(x2) : 0.0) + (double)bytes_of(wv);
        std::vector<int> eslots(RL_EPI_MAX_PTRS, -1);
        {
            Step tmp;
            st = bind_chain(chain, tmp, out_layout, bytes);
            if (st != RL_OK) return st;
            for (int i = 0; i < RL_EPI_MAX_PTRS; ++i) eslots[i] = tmp.slot[SL_E0 + i];
        }
        int cin_buf = -1, cout_buf = -1, hout_buf = -1, ybuf = -1;
        if (gates) {
            const OpNode &go = g.ops[ops.back()];
            st = need(go.in[1], L_NATIVE, cin_buf);
            if (st != RL_OK) return st;
            cout_buf = out_buf(go.out[0], L_NATIVE);
            hout_buf = out_buf(go.out[1], L_NATIVE);
            bytes += 2.0 * bytes_of(go.in[1]) + bytes_of(go.out[1]);
        } else {
            p.y_dtype = T(vout).dtype;
            ybuf = out_buf(vout, out_layout);
            bytes += (double)bytes_of(vout);
        }
        p.epi = chain.epi;
        int part_buf = -1;
        if (il.avec && !il.lp && !gates && x2 < 0 && !stem) {
            const KSlices c = k_slices(il.tile, in_dt, p.M, p.N, p.K);
            if (c.splits > 1) {
                il.splits = c.splits;
                p.splits = c.splits; p.split_tiles = c.per;
                plan.spent |= c.tiles > 64;
                part_buf = new_ws((size_t)il.splits * p.M * p.N * 4);
                bytes += 2.0 * il.splits * p.M * (double)p.N * 4;
            }
        }
        static const char *tile_names[] = {"128x128", "128x64", "64x64", "256x128"};
        std::string kname = (ov ? std::string("igemm_") + op_name(an.kind) + "_" : std::string(akind == RL_OP_CONV2D ? "igemm_conv2d_" : "igemm_dense_")) + (in_dt == RL_BF16 ? "bf16_" : "f32_") +
                            (il.c64 ? "3x3_c64" : il.ws ? "128x64_ws" : il.big ? "256x256" : tile_names[il.tile]) + (il.c64 || il.ws ? "" : il.run ? "_run" : il.lp ? "_lp" : il.avec ? (il.dma ? (il.taps ? "_dma_taps" : "_dma") : "") : "_gather") + (gates ? "_gates" : "") +
                            (il.splits > 1 ? "_splitk" : "");
        if (il.direct) {
            const char *reads[] = {"", "_planes", "_any"};
            const std::string tl = std::to_string(il.direct_tile);
            kname = kname.substr(0, kname.find(tile_names[il.tile])) + tl + "x" + (gates ? std::to_string(4 * il.direct_units) : tl) + "_direct" + reads[il.direct - 1] + (gates ? "_gates" : il.direct_slices > 1 ? "_kwaves" : "");
        }
        Step &s = add_step(S_IGEMM, std::string(op_name(an.kind)) + "#" + std::to_string(ops[ai]), kname);
        s.group = gi;
        s.ig = p; s.il = il;
        s.stem = stem ? 1 : 0;
        s.stem_kh = stem ? pack.KH : 0;
        s.slot[SL_X] = xbuf; s.slot[SL_X2] = x2buf; s.slot[SL_W] = bound(wv); s.slot[SL_Y] = ybuf;
        for (int i = 0; i < RL_EPI_MAX_PTRS; ++i) s.slot[SL_E0 + i] = eslots[i];
        s.slot[SL_CIN] = cin_buf; s.slot[SL_COUT] = cout_buf; s.slot[SL_HOUT] = hout_buf;
        s.slot[SL_PART] = part_buf;
        s.flops = flops;
        s.bytes = bytes;
        return RL_OK;
    }

    // ---- anchor-less injective groups ---------------------------------------
    rl_status plan_eltwise(int gi, const std::vector<int> &ops)
    {
        std::set<int> gset(ops.begin(), ops.end());
        const OpNode &first = g.ops[ops[0]];
        const int start = first.in[0];
        Chain chain;
        rl_status st = build_chain(ops, 0, ops.size(), start, gset, chain);
        if (st != RL_OK) return st;
        const int vout = chain.last_value;
        const rl_type &ot = T(vout);
        int layout = L_NATIVE;
        if (ot.rank == 4 && !layout_free(vout) && (chain.bias_axis < 0 || chain.bias_axis == 1) && phys[L_NATIVE][start] < 0 &&
            !out_set.count(vout))
            layout = L_NHWC;
        int xbuf;
        st = need(start, layout, xbuf);
        if (st != RL_OK) return st;
        EltwiseParams e{};
        e.x_dtype = T(start).dtype;
        e.y_dtype = ot.dtype;
        e.n = numel(ot);
        e.ch_inner = 1; e.ch_count = 1;
        if (chain.bias_axis >= 0) {
            if (layout == L_NHWC) { e.ch_inner = 1; e.ch_count = (int)ot.dims[1]; }
            else {
                int64_t inner = 1;
                for (int d = chain.bias_axis + 1; d < ot.rank; ++d) inner *= ot.dims[d];
                e.ch_inner = inner; e.ch_count = (int)ot.dims[chain.bias_axis];
            }
        }
        double bytes = (double)bytes_of(start) + (double)bytes_of(vout);
        Step tmp;
        st = bind_chain(chain, tmp, layout, bytes);
        if (st != RL_OK) return st;
        int ybuf = out_buf(vout, layout);
        e.epi = chain.epi;
        Step &s = add_step(S_ELTWISE, "eltwise#" + std::to_string(ops[0]), "eltwise_chain");
        s.group = gi;
        s.el = e;
        s.slot[SL_X] = xbuf; s.slot[SL_Y] = ybuf;
        for (int i = 0; i < RL_EPI_MAX_PTRS; ++i) s.slot[SL_E0 + i] = tmp.slot[SL_E0 + i];
        s.flops = (double)e.n * chain.epi.n_ops;
        s.bytes = bytes;
        return RL_OK;
    }

    rl_status plan_pool(int gi, int oi)
    {
        const OpNode &o = g.ops[oi];
        const rl_type &xt = T(o.in[0]), &ot = T(o.out[0]);
        int xbuf;
        rl_status st = need(o.in[0], L_NHWC, xbuf);
        if (st != RL_OK) return st;
        PoolParams p{};
        p.dtype = xt.dtype;
        p.N = (int)xt.dims[0]; p.C = (int)xt.dims[1]; p.H = (int)xt.dims[2]; p.W = (int)xt.dims[3];
        p.OH = (int)ot.dims[2]; p.OW = (int)ot.dims[3];
        bool mx = o.kind == RL_OP_MAXPOOL2D;
        if (mx) {
            p.KH = o.attrs.kernel[0]; p.KW = o.attrs.kernel[1]; p.sh = o.attrs.stride[0]; p.sw = o.attrs.stride[1];
            p.ph = o.attrs.pad[0]; p.pw = o.attrs.pad[1];
        }
        int ybuf = out_buf(o.out[0], L_NHWC);
        Step &s = add_step(mx ? S_MAXPOOL : S_GAVG, std::string(op_name(o.kind)) + "#" + std::to_string(oi), mx ? "maxpool_nhwc" : "gavgpool_nhwc");
        s.group = gi;
        s.po = p;
        s.slot[SL_X] = xbuf; s.slot[SL_Y] = ybuf;
        s.bytes = (double)bytes_of(o.in[0]) + (double)bytes_of(o.out[0]);
        s.flops = (double)numel(ot) * (mx ? p.KH * p.KW : p.H * p.W);
        return RL_OK;
    }

    rl_status plan_flatten(int oi)
    {
        const OpNode &o = g.ops[oi];
        int buf;
        rl_status st = need(o.in[0], L_NATIVE, buf);      // row-major order of the Shape is what flatten keeps
        if (st != RL_OK) return st;
        set_phys(o.out[0], L_NATIVE, buf);                // zero-copy alias
        return RL_OK;
    }

    // A change of layout (a permutation of the axes).  Rank-4 values live channel-last inside convolution, pool and
    // elementwise groups, so the two permutations between channel-first and channel-last Shapes are the other
    // view of storage that exists anyway: the result aliases it.  A permutation that keeps a prefix of the axes
    // and exchanges two blocks behind it is a batched transposition (LDS-tiled kernel); the rest gathers.
    rl_status plan_layout(int gi, int oi)
    {
        const OpNode &o = g.ops[oi];
        const int x = o.in[0], y = o.out[0];
        const rl_type &xt = T(x), &yt = T(y);
        const int r = xt.rank;
        const int32_t *pm = o.attrs.perm;
        bool ident = true;
        for (int i = 0; i < r; ++i) ident &= pm[i] == i;
        const bool to_last = r == 4 && pm[0] == 0 && pm[1] == 2 && pm[2] == 3 && pm[3] == 1;
        const bool to_first = r == 4 && pm[0] == 0 && pm[1] == 3 && pm[2] == 1 && pm[3] == 2;
        int buf;
        if (ident || (to_last && layout_free(x)) || (to_first && layout_free(y))) {     // same order in memory
            rl_status st = need(x, L_NATIVE, buf);
            if (st != RL_OK) return st;
            set_phys(y, L_NATIVE, buf);
            return RL_OK;
        }
        if (to_last && phys[L_NHWC][x] >= 0) { set_phys(y, L_NATIVE, phys[L_NHWC][x]); return RL_OK; }
        if (to_first) {
            rl_status st = need(x, L_NATIVE, buf);
            if (st != RL_OK) return st;
            set_phys(y, L_NHWC, buf);               // a consumer that wants y in Shape order gets the transposition then
            return RL_OK;
        }
        rl_status st = need(x, L_NATIVE, buf);
        if (st != RL_OK) return st;
        // identity prefix of length a, then blocks [a, a+R) and [a+R, r) exchanged?
        int a = 0;
        while (a < r && pm[a] == a) ++a;
        int split = -1;                             // first axis of the block that moves to the front
        if (a < r) {
            split = pm[a];
            bool ok = split > a;
            for (int i = a; i < r && ok; ++i) ok = pm[i] == (i - a + split < r ? i - a + split : i - a + split - r + a);
            if (!ok) split = -1;
        }
        const int ybuf = out_buf(y, L_NATIVE);
        if (split > 0) {
            int64_t outer = 1, R = 1, Q = 1;
            for (int i = 0; i < a; ++i) outer *= xt.dims[i];
            for (int i = a; i < split; ++i) R *= xt.dims[i];
            for (int i = split; i < r; ++i) Q *= xt.dims[i];
            if (outer <= 65535 && (R + 31) / 32 <= 65535 && Q <= 0x7fffffff && R <= 0x7fffffff) {
                Step &s = add_step(S_TO_NHWC, "layout_transform#" + std::to_string(oi), "transpose_tiled");
                s.group = gi;
                s.t_dtype = xt.dtype; s.t_N = (int)outer; s.t_C = (int)R; s.t_P = (int)Q;
                s.slot[SL_X] = buf; s.slot[SL_Y] = ybuf;
                s.bytes = 2.0 * bytes_of(x);
                if (to_last) phys[L_NHWC][x] = ybuf;     // the result doubles as the operand's channel-last form
                return RL_OK;
            }
        }
        PermuteParams pe{};
        pe.dtype = xt.dtype; pe.rank = r; pe.n = numel(xt);
        int64_t xs[RL_MAX_RANK];
        int64_t acc = 1;
        for (int i = r - 1; i >= 0; --i) { xs[i] = acc; acc *= xt.dims[i]; }
        for (int k = 0; k < r; ++k) { pe.ydims[k] = (int32_t)yt.dims[k]; pe.xstride[k] = xs[pm[k]]; }
        for (int k = 0; k < r; ++k) if (yt.dims[k] > 0x7fffffff) return fail(RL_ERR_UNSUPPORTED, "layout_transform: axis too long");
        Step &s = add_step(S_PERMUTE, "layout_transform#" + std::to_string(oi), "permute_gather");
        s.group = gi;
        s.pe = pe;
        s.slot[SL_X] = buf; s.slot[SL_Y] = ybuf;
        s.bytes = 2.0 * bytes_of(x);
        return RL_OK;
    }

    rl_status plan_gates(int gi, int oi)
    {
        const OpNode &o = g.ops[oi];
        int zbuf, cbuf;
        rl_status st = need(o.in[0], L_NATIVE, zbuf);
        if (st != RL_OK) return st;
        st = need(o.in[1], L_NATIVE, cbuf);
        if (st != RL_OK) return st;
        GatesParams p{};
        p.B = (int)T(o.in[1]).dims[0]; p.H = (int)T(o.in[1]).dims[1];
        p.h_dtype = T(o.out[1]).dtype;
        int cob = out_buf(o.out[0], L_NATIVE), hob = out_buf(o.out[1], L_NATIVE);
        Step &s = add_step(S_GATES, "lstm_gates#" + std::to_string(oi), "lstm_gates");
        s.group = gi;
        s.ga = p;
        s.slot[SL_X] = zbuf; s.slot[SL_CIN] = cbuf; s.slot[SL_COUT] = cob; s.slot[SL_HOUT] = hob;
        s.bytes = (double)bytes_of(o.in[0]) + 2.0 * bytes_of(o.in[1]) + bytes_of(o.out[1]);
        s.flops = 30.0 * p.B * p.H;
        return RL_OK;
    }

    // ---- partial derivatives of the contractions --------------------------------
    // Each is again a contraction C[m, n] = sum_k A[m, k] Wp[n, k] once its operands are looked at the right way round:
    //   dense_grad_x   m = batch row,       n = input feature k',  k = output feature:   A = dy,            Wp[k'][n] = W[n][k']
    //   dense_grad_w   m = output feature,  n = input feature,     k = batch row:        A[n][m] = dy[m][n], Wp[k'][m] = x[m][k']
    //   conv2d_grad_x  m = input pixel,     n = input channel,     k = (tap, out chan.): A = dy with stride-1 zeros between its
    //                  pixels and a border of K-1-pad, Wp = w with taps reversed and channel roles exchanged
    //   conv2d_grad_w  m = (in chan., tap), n = output channel,    k = (out pixel, image): A = x read with channel and image
    //                  exchanged and taps `stride` apart, Wp[o][(i, j), n] = dy[n][o][i][j]
    // A is read in place through the element-gather kernel's strides; Wp is gathered once into K-contiguous rows: at
    // prepack time when it comes from a param, by a step of the plan when it comes from an activation.
    rl_status plan_grad(int gi, int oi)
    {
        const OpNode &o = g.ops[oi];
        const int va = o.in[0], vb = o.in[1], vy = o.out[0];
        const rl_type &ta = T(va), &tb = T(vb), &ty = T(vy);
        const int dt = ta.dtype;
        const int KV = kv_of(dt);
        IgemmParams p{};
        GatherPack gp{};
        p.in_dtype = dt; p.y_dtype = ty.dtype;
        gp.dtype = dt;
        if (numel(ta) >= ((int64_t)1 << 31) || numel(tb) >= ((int64_t)1 << 31) || numel(ty) >= ((int64_t)1 << 31))
            return fail(RL_ERR_UNSUPPORTED, std::string(op_name(o.kind)) + ": tensor too large");
        // With respect to the first operand, through weights that are a param of their own: a dense, or a stride-1 conv2d
        // with reversed taps and exchanged channel roles, of dy; planned like the forward operator, onto its kernels.
        if (g.values[vb].role == ROLE_PARAM && consumers[vb].size() == 1 && !plan.packs.count(vb) && !plan.opts.no_grad_fwd) {
            AnchorView ov{};
            ov.gp.dtype = dt;
            if (o.kind == RL_OP_DENSE_GRAD_X) {
                const int N = (int)ta.dims[1], K = (int)tb.dims[1];
                ov.kind = RL_OP_DENSE; ov.N = K; ov.KH = ov.KW = 1;
                ov.gp.R = K; ov.gp.T = 1; ov.gp.TW = 1; ov.gp.Cq = N; ov.gp.s_row = 1; ov.gp.s_c = K;
                return plan_anchor(gi, std::vector<int>{oi}, &ov);
            }
            if (o.kind == RL_OP_CONV2D_GRAD_X && o.attrs.stride[0] == 1 && o.attrs.stride[1] == 1) {
                const int O = (int)ta.dims[1], C = (int)tb.dims[1], KH = (int)tb.dims[2], KW = (int)tb.dims[3];
                if (o.attrs.pad[0] > KH - 1 || o.attrs.pad[1] > KW - 1) return fail(RL_ERR_UNSUPPORTED, "conv2d_grad_x: padding larger than the kernel");
                ov.kind = RL_OP_CONV2D; ov.N = C; ov.KH = KH; ov.KW = KW; ov.ph = KH - 1 - o.attrs.pad[0]; ov.pw = KW - 1 - o.attrs.pad[1];
                ov.gp.R = C; ov.gp.T = KH * KW; ov.gp.TW = KW; ov.gp.Cq = O;
                ov.gp.s_row = (int64_t)KH * KW; ov.gp.s_c = (int64_t)C * KH * KW; ov.gp.s_ti = -KW; ov.gp.s_tj = -1; ov.gp.base = (int64_t)KH * KW - 1;
                return plan_anchor(gi, std::vector<int>{oi}, &ov);
            }
            // At a stride: the same stride-1 convolution of dy spread out with zeros (a step of its own writes that
            // tensor; three of four products are with zeros, on kernels that are many times faster than the gather).
            if (o.kind == RL_OP_CONV2D_GRAD_X && o.attrs.stride[0] == o.attrs.stride[1] && o.attrs.stride[0] > 1 &&
                ((ta.dims[1] * (int64_t)dtype_size(dt)) % 16 == 0 || (!plan.lean && moves_to_rows(ta)))) {
                const int Nb = (int)ta.dims[0], O = (int)ta.dims[1], OH = (int)ta.dims[2], OW = (int)ta.dims[3];
                const int C = (int)tb.dims[1], KH = (int)tb.dims[2], KW = (int)tb.dims[3], H = (int)ty.dims[2], W = (int)ty.dims[3];
                const int sd = o.attrs.stride[0];
                if (o.attrs.pad[0] > KH - 1 || o.attrs.pad[1] > KW - 1) return fail(RL_ERR_UNSUPPORTED, "conv2d_grad_x: padding larger than the kernel");
                const int Hd = H + 2 * o.attrs.pad[0] - KH + 1, Wd = W + 2 * o.attrs.pad[1] - KW + 1;
                // channels of dy that are no whole vectors: rows padded with zeros (60 drawn backward passes 0.39 of the gather's time, the
                // worst 0.85: 6x44x38x38 -> 198 3x3/2 bf16 235 -> 33 us; the extra workspace is not for the smallest form of a plan)
                const int ld = (int)round_up(O, KV);
                const size_t dbytes = (size_t)Nb * Hd * Wd * ld * dtype_size(dt);
                if (Hd >= (OH - 1) * sd + 1 && Wd >= (OW - 1) * sd + 1 && dbytes < ((size_t)1 << 31)) {
                    int src, rows = O;
                    if (ld != O) plan.spent = true;
                    rl_status st = ld == O ? need(va, L_NHWC, src) : need_rows(gi, va, src, rows);
                    if (st != RL_OK) return st;
                    const int dil = new_ws(dbytes);
                    Step &ds = add_step(S_DILATE, std::string(op_name(o.kind)) + "#" + std::to_string(oi) + ".spread", "dilate_nhwc");
                    ds.group = gi;
                    ds.t_N = Nb; ds.t_C = (int)(ld * dtype_size(dt)); ds.st_H = OH; ds.st_W = OW; ds.st_Hp = Hd; ds.st_Wp = Wd; ds.st_ph = sd;
                    ds.slot[SL_X] = src; ds.slot[SL_Y] = dil;
                    ds.bytes = (double)bytes_of(va) + (double)dbytes;
                    ov.kind = RL_OP_CONV2D; ov.N = C; ov.KH = KH; ov.KW = KW; ov.ph = KH - 1 - o.attrs.pad[0]; ov.pw = KW - 1 - o.attrs.pad[1];
                    ov.gp.R = C; ov.gp.T = KH * KW; ov.gp.TW = KW; ov.gp.Cq = O;
                    ov.gp.s_row = (int64_t)KH * KW; ov.gp.s_c = (int64_t)C * KH * KW; ov.gp.s_ti = -KW; ov.gp.s_tj = -1; ov.gp.base = (int64_t)KH * KW - 1;
                    if (ld != O) { ov.xC = ov.gp.Cq = ld; ov.gp.Creal = O; }
                    ov.xbuf = dil; ov.xH = Hd; ov.xW = Wd;
                    st = plan_anchor(gi, std::vector<int>{oi}, &ov);
                    if (st != RL_OK) return st;
                    for (size_t k = plan.steps.size(); k-- > 0;)
                        if (plan.steps[k].kind == S_IGEMM) { plan.steps[k].flops *= (double)O / (double)((int64_t)sd * sd * ld); break; }     // the zeros are no work
                    return RL_OK;
                }
            }
        }
        if (o.kind == RL_OP_DENSE_GRAD_W && tn_ok(o)) return plan_tn(gi, oi);
        p.C = 1; p.H = p.W = p.KH = p.KW = p.OH = p.OW = p.OHW = 1; p.sh = p.sw = 1;
        if (o.kind == RL_OP_DENSE_GRAD_X) {
            const int M = (int)ta.dims[0], N = (int)ta.dims[1], K = (int)tb.dims[1];
            p.M = M; p.N = K; p.K = N; p.C = N;
            p.xs_n = N; p.xs_c = 1;
            gp.R = K; gp.T = 1; gp.TW = 1; gp.Cq = N; gp.s_row = 1; gp.s_c = K;
        } else if (o.kind == RL_OP_DENSE_GRAD_W) {
            const int M = (int)ta.dims[0], N = (int)ta.dims[1], K = (int)tb.dims[1];
            p.M = N; p.N = K; p.K = M; p.C = M;
            p.xs_n = 1; p.xs_c = N;
            gp.R = K; gp.T = 1; gp.TW = 1; gp.Cq = M; gp.s_row = 1; gp.s_c = K;
        } else if (o.kind == RL_OP_CONV2D_GRAD_X) {
            // dy[N,O,OH,OW], w[O,C,KH,KW] -> dx[N,C,H,W]
            const int Nb = (int)ta.dims[0], O = (int)ta.dims[1], OH = (int)ta.dims[2], OW = (int)ta.dims[3];
            const int C = (int)tb.dims[1], KH = (int)tb.dims[2], KW = (int)tb.dims[3], H = (int)ty.dims[2], W = (int)ty.dims[3];
            if (o.attrs.stride[0] != o.attrs.stride[1]) return fail(RL_ERR_UNSUPPORTED, "conv2d_grad_x: strides must agree");
            if (o.attrs.pad[0] > KH - 1 || o.attrs.pad[1] > KW - 1) return fail(RL_ERR_UNSUPPORTED, "conv2d_grad_x: padding larger than the kernel");
            if ((int64_t)Nb * H * W > 0x7fffffff) return fail(RL_ERR_UNSUPPORTED, "conv2d_grad_x too large");
            p.M = Nb * H * W; p.N = C; p.K = O * KH * KW; p.C = O;
            p.H = OH; p.W = OW; p.KH = KH; p.KW = KW; p.OH = H; p.OW = W; p.OHW = H * W;
            p.sh = p.sw = 1; p.ph = KH - 1 - o.attrs.pad[0]; p.pw = KW - 1 - o.attrs.pad[1];
            p.in_dil_m1 = o.attrs.stride[0] - 1;
            p.xs_n = (int64_t)O * OH * OW; p.xs_c = (int64_t)OH * OW; p.xs_h = OW; p.xs_w = 1;
            p.ys_n = (int64_t)C * H * W; p.ys_p = 1; p.ys_c = (int64_t)H * W;
            // Wp[c][(a', b'), o] = w[o][c][KH-1-a'][KW-1-b']
            gp.R = C; gp.T = KH * KW; gp.TW = KW; gp.Cq = O;
            gp.s_row = (int64_t)KH * KW; gp.s_c = (int64_t)C * KH * KW; gp.s_ti = -KW; gp.s_tj = -1; gp.base = (int64_t)KH * KW - 1;
        } else {
            // dy[N,O,OH,OW], x[N,C,H,W] -> dw[O,C,KH,KW]
            const int Nb = (int)ta.dims[0], O = (int)ta.dims[1], OH = (int)ta.dims[2], OW = (int)ta.dims[3];
            const int C = (int)tb.dims[1], H = (int)tb.dims[2], W = (int)tb.dims[3], KH = (int)ty.dims[2], KW = (int)ty.dims[3];
            if (o.attrs.stride[0] != o.attrs.stride[1]) return fail(RL_ERR_UNSUPPORTED, "conv2d_grad_w: strides must agree");
            // bf16 batches of 64 whose operands are both channel-first still: transposed to images-last; once one of them is held
            // channel-last, the rows are contracted as they are
            const bool rows_held = phys[L_NHWC][va] >= 0 || phys[L_NHWC][vb] >= 0;
            if (rows_held && tn_ok(o)) return plan_tn(gi, oi);
            if (dt == RL_BF16 && conv_wgrad_ok(Nb, O, C, KH, KW, o.attrs.stride[0]) && o.attrs.pad[0] < KH && o.attrs.pad[1] < KW &&
                bytes_of(va) < ((size_t)1 << 31) && bytes_of(vb) < ((size_t)1 << 31) && !plan.opts.no_wgrad)
                return plan_wgrad(gi, oi);
            if ((int64_t)Nb * OH * OW > 0x7ffffff0) return fail(RL_ERR_UNSUPPORTED, "conv2d_grad_w too large");
            if (tn_ok(o)) return plan_tn(gi, oi);
            p.M = C * KH * KW; p.N = O; p.K = Nb * OH * OW; p.C = Nb;
            p.H = H; p.W = W; p.KH = OH; p.KW = OW; p.OH = KH; p.OW = KW; p.OHW = KH * KW;
            p.sh = p.sw = 1; p.ph = o.attrs.pad[0]; p.pw = o.attrs.pad[1];
            p.tap_dil_m1 = o.attrs.stride[0] - 1;
            p.xs_n = (int64_t)H * W; p.xs_c = (int64_t)C * H * W; p.xs_h = W; p.xs_w = 1;      // "image" = channel c, "channel" = image n
            p.ys_n = (int64_t)KH * KW; p.ys_p = 1; p.ys_c = (int64_t)C * KH * KW;               // dw[o][c][a][b] at n*ys_c + m
            // Wp[o][(i, j), n] = dy[n][o][i][j]
            gp.R = O; gp.T = OH * OW; gp.TW = OW; gp.Cq = Nb;
            gp.s_row = (int64_t)OH * OW; gp.s_c = (int64_t)O * OH * OW; gp.s_ti = OW; gp.s_tj = 1;
        }
        if (o.kind == RL_OP_DENSE_GRAD_X || o.kind == RL_OP_DENSE_GRAD_W) { p.ys_n = p.N; p.ys_p = p.N; p.ys_c = 1; }
        p.K1 = p.K;
        // A small dense weight gradient (below tn_ok's line) of a backward pass, whose dy others read too: dy and x as they lie, on the kernel
        // without LDS tiles.  The gather packs x first and reads dy element by element on a few 64x64 tiles: of 90 drawn backward passes some 60 go
        // this way, at 0.47 of their time (514 x 53 x 59 bf16 36 -> 9.5 us, 14 x 128 x 88 18.3 -> 7.4).  Not from 25 K steps a wave on, where
        // the gather cuts K over workgroups (4071 x 21 x 16 f32 19.7 against 21.9); an operator alone in its plan keeps the packed operand.
        if (o.kind == RL_OP_DENSE_GRAD_W && consumers[va].size() > 1 && (double)p.M * p.N * p.K < 4e6 && !plan.opts.no_direct && g.values[va].role != ROLE_PARAM && g.values[vb].role != ROLE_PARAM && bytes_of(va) < ((size_t)1 << 31) &&
            bytes_of(vb) < ((size_t)1 << 31) && (int64_t)p.M * p.N < ((int64_t)1 << 31)) {
            double us = 0.0;
            const Direct form = direct_form(dt, p.M, p.N, p.K, DIRECT_ANY, OTHER_GATHER, false, 0.0, false, 1, false, false, false, 0.0, &us);
            const int per_step = KV * (64 / std::max(form.tile, 1));
            if (form.tile && (p.K + per_step - 1) / per_step <= 24 * form.slices) {
                int a, b;
                rl_status st = need(va, L_NATIVE, a);
                if (st == RL_OK) st = need(vb, L_NATIVE, b);
                if (st != RL_OK) return st;
                p.Kp = p.N; p.w_frag = 2;
                p.x_bytes = (uint32_t)bytes_of(va); p.w_bytes = (uint32_t)bytes_of(vb); p.y_bytes = (uint32_t)std::min(bytes_of(vy), ((size_t)1 << 31) - 1);
                p.ts_h = p.xs_h; p.ts_w = p.xs_w; p.seg_stride = 64;
                make_fast_div(1, p.div_ohw_mul, p.div_ohw_sh);
                make_fast_div(1, p.div_ow_mul, p.div_ow_sh);
                make_fast_div((uint32_t)p.C, p.div_c_mul, p.div_c_sh);
                make_fast_div(1, p.div_kw_mul, p.div_kw_sh);
                const int y = out_buf(vy, L_NATIVE);
                const std::string tl = std::to_string(form.tile);
                Step &s = add_step(S_IGEMM, std::string(op_name(o.kind)) + "#" + std::to_string(oi),
                                   std::string("igemm_") + op_name(o.kind) + (dt == RL_BF16 ? "_bf16_" : "_f32_") + tl + "x" + tl + "_direct_columns" + (form.slices > 1 ? "_kwaves" : ""));
                s.group = gi;
                s.ig = p;
                s.il.direct = 1 + DIRECT_ANY; s.il.direct_tile = form.tile; s.il.direct_slices = form.slices;
                s.slot[SL_X] = a; s.slot[SL_W] = b; s.slot[SL_Y] = y;
                s.flops = 2.0 * p.M * (double)p.N * p.K;
                s.bytes = (double)bytes_of(va) + (double)bytes_of(vb) + (double)bytes_of(vy);
                return RL_OK;
            }
        }
        p.Kp = (int)round_up(p.K, KV);
        gp.Kp = p.Kp;
        p.ts_h = p.xs_h; p.ts_w = p.xs_w; p.seg_stride = 64;
        make_fast_div((uint32_t)p.OHW, p.div_ohw_mul, p.div_ohw_sh);
        make_fast_div((uint32_t)p.OW, p.div_ow_mul, p.div_ow_sh);
        const size_t lim = (size_t)1 << 31;
        const size_t wbytes = (size_t)gp.R * gp.Kp * dtype_size(dt);
        if (wbytes >= lim) return fail(RL_ERR_UNSUPPORTED, std::string(op_name(o.kind)) + ": operand too large");
        p.x_bytes = (uint32_t)std::min(bytes_of(va), lim - 1);
        p.w_bytes = (uint32_t)wbytes;
        p.y_bytes = (uint32_t)std::min(bytes_of(vy), lim - 1);

        int abuf, wbuf;
        rl_status st;
        // which of the two operands is A and which is gathered into Wp: dy is A except for conv2d_grad_w, where x is
        int a_val = va, w_val = vb;
        if (o.kind == RL_OP_CONV2D_GRAD_W) { a_val = vb; w_val = va; }
        st = need(a_val, L_NATIVE, abuf);
        if (st != RL_OK) return st;
        if (g.values[w_val].role == ROLE_PARAM && consumers[w_val].size() == 1) {     // a param with other uses keeps its own layout for them
            PackSpec pack;
            pack.dtype = dt; pack.gather = 1; pack.gp = gp; pack.bytes = wbytes; pack.Kp = gp.Kp; pack.perm_block = -3;
            auto it = plan.packs.find(w_val);
            if (it != plan.packs.end()) return fail(RL_ERR_UNSUPPORTED, "one param needs two different kernel-native layouts");
            plan.packs[w_val] = pack;
            wbuf = bound(w_val);
        } else {
            int src;
            st = need(w_val, L_NATIVE, src);
            if (st != RL_OK) return st;
            wbuf = new_ws(wbytes);
            Step &ps = add_step(S_PACK, std::string(op_name(o.kind)) + "#" + std::to_string(oi) + ".operand", "pack_gather");
            ps.group = gi;
            ps.gp = gp;
            ps.slot[SL_X] = src; ps.slot[SL_Y] = wbuf;
            ps.bytes = (double)bytes_of(w_val) + (double)wbytes;
        }
        const int ybuf = out_buf(vy, L_NATIVE);
        IgemmLaunch il{};
        il.tile = TILE_64x64;                         // element gather: any strides, any counts
        // few tiles and a long K (a weight gradient contracts over every pixel of the batch): K split over workgroups
        int part_buf = -1;
        if (!plan.opts.no_splitk) {
            const int64_t tiles = (int64_t)((p.M + 63) / 64) * ((p.N + 63) / 64);
            const int nk = (p.Kp + 8 * KV - 1) / (8 * KV);
            const int want = (int)std::min<int64_t>(std::min<int64_t>(64, 512 / std::max<int64_t>(tiles, 1)), nk / 4);
            if (tiles <= 128 && want >= 2 && (int64_t)want * p.M * p.N * 4 < (int64_t)1 << 28) {
                const int per = (nk + want - 1) / want;
                il.splits = (nk + per - 1) / per;
                p.splits = il.splits; p.split_tiles = per;
                part_buf = new_ws((size_t)il.splits * p.M * p.N * 4);
            }
        }
        Step &s = add_step(S_IGEMM, std::string(op_name(o.kind)) + "#" + std::to_string(oi),
                           std::string("igemm_") + op_name(o.kind) + (dt == RL_BF16 ? "_bf16" : "_f32") + "_64x64_gather");
        s.group = gi;
        s.ig = p; s.il = il;
        s.slot[SL_X] = abuf; s.slot[SL_W] = wbuf; s.slot[SL_Y] = ybuf; s.slot[SL_PART] = part_buf;
        if (il.splits > 1) s.kernel += "_splitk";
        s.flops = 2.0 * p.M * (double)p.N * p.K / (double)((p.in_dil_m1 + 1) * (p.in_dil_m1 + 1));     // the zeros between dy's pixels are no work
        s.bytes = (double)bytes_of(va) + (double)bytes_of(vb) + (double)bytes_of(vy);
        return RL_OK;
    }

    // Whether need_rows' change of layout of a tensor of rank 4 fits the grid of its launch (launch_move): images and, but for whole vectors
    // either way, tiles of channels in two dimensions of at most 65535.
    static bool moves_to_rows(const rl_type &t)
    {
        const int64_t KV = kv_of(t.dtype), C = t.dims[1], P = t.dims[2] * t.dims[3];
        return C % KV != 0 ? t.dims[0] <= 65535 && (round_up(C, KV) + 63) / 64 <= 65535 : P == 1 || P % KV == 0 || (t.dims[0] <= 65535 && (C + 31) / 32 <= 65535);
    }

    // Rows of value v with its channels (features) fastest, each a whole number of 16-byte vectors long: v's own storage where
    // it has that form, else a copy padded with zeros by a step of the plan.  ld: elements per row.
    rl_status need_rows(int gi, int v, int &buf, int &ld)
    {
        const rl_type &t = T(v);
        const int KV = kv_of(t.dtype), C = (int)t.dims[1];
        ld = (int)round_up(C, KV);
        if (ld == C) return need(v, t.rank == 4 ? L_NHWC : L_NATIVE, buf);
        auto it = padded_rows.find(v);
        if (it != padded_rows.end()) { buf = it->second; return RL_OK; }
        const int64_t P = t.rank == 4 ? t.dims[2] * t.dims[3] : 1;
        const bool cl = t.rank == 2 || phys[L_NHWC][v] >= 0;
        int src;
        rl_status st = need(v, t.rank == 4 && cl ? L_NHWC : L_NATIVE, src);
        if (st != RL_OK) return st;
        buf = new_ws((size_t)t.dims[0] * P * ld * dtype_size(t.dtype));
        Step &s = add_step(cl ? S_PACK : S_PAD_NHWC, "padded rows", cl ? "pack_gather" : "nchw_to_nhwc_padded");
        s.group = gi;
        if (cl) {
            s.gp.dtype = t.dtype; s.gp.R = (int)(t.dims[0] * P); s.gp.Kp = ld; s.gp.T = s.gp.TW = 1; s.gp.Cq = C; s.gp.s_row = C; s.gp.s_c = 1;
        } else {
            s.t_dtype = t.dtype; s.t_N = (int)t.dims[0]; s.t_C = C; s.t_P = (int)P; s.st_W = ld;
        }
        s.slot[SL_X] = src; s.slot[SL_Y] = buf;
        s.bytes = (double)bytes_of(v) + (double)t.dims[0] * P * ld * dtype_size(t.dtype);
        padded_rows[v] = buf;
        return RL_OK;
    }

    // Whether a weight gradient runs on the kernel that contracts over the rows of both operands (igemm_tn.hip).  The element
    // gather it replaces reads single elements and needs its operand packed first; below these sizes its few K tiles are not
    // what the call's time is.
    bool tn_ok(const OpNode &o) const
    {
        const int va = o.in[0], vb = o.in[1];
        const rl_type &ta = T(va), &tb = T(vb);
        if (plan.lean || plan.opts.no_wgrad || g.values[va].role == ROLE_PARAM || g.values[vb].role == ROLE_PARAM) return false;
        const bool conv = o.kind == RL_OP_CONV2D_GRAD_W;
        const int64_t P = conv ? ta.dims[0] * ta.dims[2] * ta.dims[3] : ta.dims[0], T_ = conv ? numel(T(o.out[0])) / (ta.dims[1] * tb.dims[1]) : 1;
        const double macs = (double)P * ta.dims[1] * tb.dims[1] * T_;
        // a convolution's backward pass, whose dy others read too (its rows are there, or their copy is shared): at any size (90 drawn ones
        // below 33 M multiply-adds take 0.51 of the gather's time, the worst 0.90: 25x12x51x51 -> 10 1x1 bf16 75 -> 26 us)
        if (macs < (conv ? 3.3e7 : 4e6) && !(conv && consumers[va].size() > 1)) return false;
        const int es = (int)dtype_size(ta.dtype), KV = kv_of(ta.dtype);
        const int64_t lda = round_up(ta.dims[1], KV), ldb = round_up(tb.dims[1], KV), lim = (int64_t)1 << 31;
        const int64_t brows = conv ? tb.dims[0] * tb.dims[2] * tb.dims[3] : P;
        return P * lda * es < lim && brows * ldb * es < lim && lda * ldb * T_ < ((int64_t)1 << 28) && ta.dims[0] <= 65535 && (!conv || (moves_to_rows(ta) && moves_to_rows(tb)));
    }

    rl_status plan_tn(int gi, int oi)
    {
        plan.spent = true;
        const OpNode &o = g.ops[oi];
        const int va = o.in[0], vb = o.in[1], vy = o.out[0];
        const rl_type &ta = T(va), &tb = T(vb), &ty = T(vy);
        const bool conv = o.kind == RL_OP_CONV2D_GRAD_W;
        const int dt = ta.dtype, es = (int)dtype_size(dt);
        TnParams p{};
        int abuf, bbuf;
        rl_status st = need_rows(gi, va, abuf, p.lda);
        if (st != RL_OK) return st;
        st = need_rows(gi, vb, bbuf, p.ldb);
        if (st != RL_OK) return st;
        p.Mout = (int)ta.dims[1]; p.Cout = (int)tb.dims[1];
        p.M = p.lda; p.C = p.ldb; p.T = 1; p.KW = 1;
        p.P = (int)ta.dims[0];
        p.H = p.W = p.OW = p.OHW = 1; p.s = 1;
        int64_t brows = p.P;
        if (conv) {
            p.OW = (int)ta.dims[3]; p.OHW = (int)(ta.dims[2] * ta.dims[3]);
            p.P = (int)(ta.dims[0] * p.OHW);
            p.H = (int)tb.dims[2]; p.W = (int)tb.dims[3];
            p.KW = (int)ty.dims[3]; p.T = (int)(ty.dims[2] * ty.dims[3]);
            p.s = o.attrs.stride[0]; p.ph = o.attrs.pad[0]; p.pw = o.attrs.pad[1];
            brows = tb.dims[0] * p.H * p.W;
            p.conv = !(p.T == 1 && p.s == 1 && p.ph == 0 && p.pw == 0);      // else output pixel p is input pixel p
        }
        p.N = p.T * p.C;
        p.a_bytes = (uint32_t)((int64_t)p.P * p.lda * es);
        p.b_bytes = (uint32_t)(brows * p.ldb * es);
        make_fast_div((uint32_t)p.OHW, p.div_ohw_mul, p.div_ohw_sh);
        make_fast_div((uint32_t)p.OW, p.div_ow_mul, p.div_ow_sh);
        // Tile and K slices by a cost in shader cycles (fitted to a sweep of both tiles over 1 to 85 slices, 64x128x28x28 bf16 and
        // 32x64x28x28 f32 through 3x3): a K tile takes `alone` cycles where a CU holds one workgroup and `share` per workgroup
        // where it holds several (three 64x64 ones fit); 4000 to start and end; 6500 for the adding launch, and the traffic of
        // the partial sums at 2200 bytes per cycle.
        const int nk = (p.P + 128 / es - 1) / (128 / es);
        int tile = 64;
        double best = 1e30;
        for (int tl : {64, 128}) {
            const int64_t tiles = (int64_t)((p.M + tl - 1) / tl) * ((p.N + tl - 1) / tl);
            const double alone = es == 2 ? (tl == 128 ? 1330 : 680) : (tl == 128 ? 4550 : 1450);
            const double share = es == 2 ? (tl == 128 ? 1330 : 390) : (tl == 128 ? 4550 : 1100);
            for (int sp = 1; sp <= std::min(nk, 512); ++sp) {
                const int per = (nk + sp - 1) / sp;
                if ((nk + per - 1) / per != sp || (sp > 1 && (int64_t)sp * p.M * p.N >= (int64_t)1 << 27)) continue;     // partial sums below 512 MB
                const double cost = per * std::max(alone, share * (double)((tiles * sp + 255) / 256)) + 4000.0 +
                                    (sp > 1 ? 6500.0 + 8.0 * sp * p.M * (double)p.N / 2200.0 : 0.0);
                if (cost < best) { best = cost; tile = tl; p.splits = sp; p.split_tiles = per; }
            }
        }
        if (p.splits < 1) return fail(RL_ERR_UNSUPPORTED, "internal: no tile for the contraction over rows");
        const int part = p.splits > 1 ? new_ws((size_t)p.splits * p.M * p.N * 4) : -1;
        const int ybuf = out_buf(vy, L_NATIVE);
        p.y_dtype = ty.dtype;
        Step &s = add_step(S_TN, std::string(op_name(o.kind)) + "#" + std::to_string(oi), std::string("igemm_") + op_name(o.kind) + (dt == RL_BF16 ? "_bf16_" : "_f32_") +
                           (tile == 128 ? "128x128" : "64x64") + "_rows" + (p.splits > 1 ? "_splitk" : ""));
        s.group = gi;
        s.tn = p; s.tn_tile = tile; s.t_dtype = dt; s.tn_cost = best;
        s.slot[SL_X] = abuf; s.slot[SL_X2] = bbuf; s.slot[SL_Y] = ybuf; s.slot[SL_PART] = part;
        s.flops = 2.0 * p.P * (double)p.Mout * p.Cout * p.T;
        s.bytes = (double)bytes_of(va) + (double)bytes_of(vb) + (double)bytes_of(vy);
        return RL_OK;
    }

    // conv2d_grad_w on bf16 batches of 64: both operands transposed so that the images are the fastest axis (two steps),
    // the contraction per output pixel and filter tap (conv_wgrad.hip), the row segments' sums added in order (a step).
    rl_status plan_wgrad(int gi, int oi)
    {
        const OpNode &o = g.ops[oi];
        const int vdy = o.in[0], vx = o.in[1], vy = o.out[0];
        const rl_type &ta = T(vdy), &tb = T(vx), &ty = T(vy);
        const int Nb = (int)ta.dims[0], O = (int)ta.dims[1], OH = (int)ta.dims[2], OW = (int)ta.dims[3];
        const int C = (int)tb.dims[1], H = (int)tb.dims[2], W = (int)tb.dims[3], KH = (int)ty.dims[2], KW = (int)ty.dims[3];
        WgradParams w{};
        w.O = O; w.C = C; w.H = H; w.W = W; w.OH = OH; w.OW = OW; w.KH = KH; w.KW = KW;
        w.s = o.attrs.stride[0]; w.ph = o.attrs.pad[0]; w.pw = o.attrs.pad[1];
        // an operand as the plan holds it (channel-last if some group already wrote or asked for that, else as declared),
        // viewed as a matrix [images][everything else] and transposed
        auto batch_last = [&](int v, int Cc, int P, int64_t &s_pix, int64_t &s_ch, int &tbuf) -> rl_status {
            int src;
            const bool cl = phys[L_NHWC][v] >= 0;
            rl_status st = need(v, cl ? L_NHWC : L_NATIVE, src);
            if (st != RL_OK) return st;
            if (cl) { s_pix = (int64_t)Cc * Nb; s_ch = Nb; }
            else { s_pix = Nb; s_ch = (int64_t)P * Nb; }
            tbuf = new_ws(bytes_of(v));
            Step &ts = add_step(S_TO_NHWC, std::string(op_name(o.kind)) + "#" + std::to_string(oi) + ".images_last", "transpose_images_last");
            ts.group = gi;
            ts.t_dtype = T(v).dtype; ts.t_N = 1; ts.t_C = Nb; ts.t_P = Cc * P;
            ts.slot[SL_X] = src; ts.slot[SL_Y] = tbuf;
            ts.bytes = 2.0 * bytes_of(v);
            return RL_OK;
        };
        int dyT, xT;
        rl_status st = batch_last(vdy, O, OH * OW, w.ys_pix, w.ys_o, dyT);
        if (st != RL_OK) return st;
        st = batch_last(vx, C, H * W, w.xs_pix, w.xs_c, xT);
        if (st != RL_OK) return st;
        w.nck = Nb / 64;
        w.n_ot = O % 128 == 0 ? O / 128 : O / 64;
        w.n_ct = C / 64;
        // one workgroup per CU (its LDS is full): as many row segments as keep the grid within one round
        const int tiles = OH * w.n_ot * w.n_ct;
        int nseg = std::max(1, std::min(OW, 256 / std::max(tiles, 1)));
        w.L = (OW + nseg - 1) / nseg;
        w.nseg = (OW + w.L - 1) / w.L;
        const int chunks = OH * w.nseg, Tt = KH * KW;
        const size_t part_bytes = (size_t)chunks * Tt * O * C * 4;
        if (part_bytes >= ((size_t)1 << 32)) return fail(RL_ERR_UNSUPPORTED, "conv2d_grad_w: partial sums too large");
        const int part = new_ws(part_bytes);
        Step &s = add_step(S_WGRAD, std::string(op_name(o.kind)) + "#" + std::to_string(oi), std::string("conv2d_grad_w_bf16_") + (O % 128 == 0 ? "128x64" : "64x64") + "_images_last");
        s.group = gi;
        s.wg = w;
        s.slot[SL_X] = xT; s.slot[SL_X2] = dyT; s.slot[SL_PART] = part;
        s.flops = 2.0 * Nb * OH * OW * (double)O * C * Tt;
        s.bytes = (double)bytes_of(vdy) + (double)bytes_of(vx) + (double)part_bytes;
        const int ybuf = out_buf(vy, L_NATIVE);
        Step &r = add_step(S_WGRAD_REDUCE, std::string(op_name(o.kind)) + "#" + std::to_string(oi) + ".segments", "wgrad_reduce");
        r.group = gi;
        r.wg = w;
        r.t_dtype = ty.dtype; r.t_N = chunks; r.t_C = Tt;
        r.slot[SL_X] = part; r.slot[SL_Y] = ybuf;
        r.bytes = (double)part_bytes + (double)bytes_of(vy);
        return RL_OK;
    }

    rl_status plan_group(int gi, std::vector<int> ops)
    {
        std::sort(ops.begin(), ops.end());
        rl_status st = check_group(g, ops, msg);
        if (st != RL_OK) return st;
        bool has_anchor = false;
        for (int o : ops) has_anchor |= is_anchor(g.ops[o].kind);
        if (has_anchor) return plan_anchor(gi, ops);
        int k0 = g.ops[ops[0]].kind;
        if (ops.size() == 1) {
            if (k0 == RL_OP_MAXPOOL2D || k0 == RL_OP_GLOBAL_AVGPOOL) return plan_pool(gi, ops[0]);
            if (k0 == RL_OP_FLATTEN) return plan_flatten(ops[0]);
            if (k0 == RL_OP_LSTM_GATES) return plan_gates(gi, ops[0]);
            if (k0 == RL_OP_LAYOUT_TRANSFORM) return plan_layout(gi, ops[0]);
            if (k0 >= RL_OP_DENSE_GRAD_X && k0 <= RL_OP_CONV2D_GRAD_W) return plan_grad(gi, ops[0]);
            if (k0 == RL_OP_CONCAT) return fail(RL_ERR_UNSUPPORTED, "concat is only implemented as the operand of a dense in its group");
        }
        return plan_eltwise(gi, ops);
    }

    rl_status run()
    {
        const int nv = (int)g.values.size();
        plan.values = g.values;
        plan.outputs = g.outputs;
        plan.err = g.err;
        plan.bound_buf.assign(nv, -1);
        phys[0].assign(nv, -1);
        phys[1].assign(nv, -1);
        out_set.insert(g.outputs.begin(), g.outputs.end());
        if (g.outputs.empty()) return fail(RL_ERR_TYPE, "graph has no output");
        consumers.assign(nv, {});
        for (size_t o = 0; o < g.ops.size(); ++o)
            for (int v : g.ops[o].in) consumers[v].push_back((int)o);
        for (int v = 0; v < nv; ++v)
            if (g.values[v].role != ROLE_OP) set_phys(v, L_NATIVE, bound(v));

        // groups: declared ones plus a singleton for every ungrouped call
        std::vector<std::vector<int>> groups = g.groups;
        std::vector<int> group_of(g.ops.size(), -1);
        for (size_t gi = 0; gi < groups.size(); ++gi)
            for (int o : groups[gi]) {
                if (o < 0 || o >= (int)g.ops.size() || group_of[o] >= 0) return fail(RL_ERR_GROUP, "an op is missing or in two groups");
                group_of[o] = (int)gi;
            }
        for (size_t o = 0; o < g.ops.size(); ++o)
            if (group_of[o] < 0) { group_of[o] = (int)groups.size(); groups.push_back({(int)o}); }

        // order groups so that producers run first; a cycle between groups is illegal
        const int ng = (int)groups.size();
        std::vector<std::set<int>> deps(ng);
        for (size_t o = 0; o < g.ops.size(); ++o)
            for (int v : g.ops[o].in) {
                int pr = g.values[v].producer;
                if (pr >= 0 && group_of[pr] != group_of[o]) deps[group_of[o]].insert(group_of[pr]);
            }
        std::vector<int> order, state(ng, 0);
        std::vector<int> key(ng);
        for (int i = 0; i < ng; ++i) key[i] = *std::min_element(groups[i].begin(), groups[i].end());
        std::vector<int> by_key(ng);
        for (int i = 0; i < ng; ++i) by_key[i] = i;
        std::sort(by_key.begin(), by_key.end(), [&](int a, int b) { return key[a] < key[b]; });
        bool cyc = false;
        std::vector<std::pair<int, std::set<int>::iterator>> stack;
        for (int root : by_key) {
            if (state[root]) continue;
            stack.push_back({root, deps[root].begin()});
            state[root] = 1;
            while (!stack.empty()) {
                auto &top = stack.back();
                if (top.second == deps[top.first].end()) {
                    state[top.first] = 2;
                    order.push_back(top.first);
                    stack.pop_back();
                } else {
                    int d = *top.second;
                    ++top.second;
                    if (state[d] == 1) { cyc = true; break; }
                    if (state[d] == 0) { state[d] = 1; stack.push_back({d, deps[d].begin()}); }
                }
            }
            if (cyc) return fail(RL_ERR_GROUP, "fusion groups depend on each other cyclically");
        }
        for (int gi : order) {
            rl_status st = plan_group(gi, groups[gi]);
            if (st != RL_OK) return st;
        }
        // every output must end up in its bound buffer in boundary order
        for (int v : g.outputs) {
            int b = bound(v);
            if (phys[L_NATIVE][v] == b) continue;
            if (phys[L_NATIVE][v] >= 0) {
                EltwiseParams e{};
                e.x_dtype = e.y_dtype = T(v).dtype;
                e.n = numel(T(v));
                e.ch_inner = 1; e.ch_count = 1;
                int src = phys[L_NATIVE][v];
                Step &s = add_step(S_ELTWISE, "copy_out", "eltwise_chain");
                s.el = e;
                s.slot[SL_X] = src; s.slot[SL_Y] = b;
                s.bytes = 2.0 * bytes_of(v);
            } else if (phys[L_NHWC][v] >= 0) {
                const rl_type &t = T(v);
                int src = phys[L_NHWC][v];
                Step &s = add_step(S_TO_NCHW, "layout_out", "nhwc_to_nchw");
                s.t_dtype = t.dtype; s.t_N = (int)t.dims[0]; s.t_C = (int)t.dims[1]; s.t_P = (int)(t.dims[2] * t.dims[3]);
                s.slot[SL_X] = src; s.slot[SL_Y] = b;
                s.bytes = 2.0 * bytes_of(v);
            } else {
                return fail(RL_ERR_TYPE, "an output is never computed");
            }
        }
        fuse_stem_pool();
        fuse_direct_store();
        pair_contractions();
        pair_gradients();
        run_weight_gradients();
        fuse_planes_store();
        pair_moves();
        chain_small_dense();
        assign_workspace();
        return RL_OK;
    }

    // A stem convolution group whose only consumer is the 3x3 / stride 2 / pad 1 max-pool group right behind it
    // runs as one kernel that pools the finished values in LDS: the full-size tensor between the two groups
    // (the largest of the whole graph) is then never written.  Same values as the two kernels, bit for bit
    // (max commutes with the bias, the ReLU and the rounding).
    void fuse_stem_pool()
    {
        if (plan.opts.no_stem_pool) return;
        for (size_t si = 0; si + 1 < plan.steps.size(); ++si) {
            Step &c = plan.steps[si];
            const Step &m = plan.steps[si + 1];
            const IgemmParams &g = c.ig;
            if (c.kind != S_IGEMM || !c.stem || !c.il.lp || m.kind != S_MAXPOOL) continue;
            const int mid = c.slot[SL_Y];
            if (mid < 0 || m.slot[SL_X] != mid || plan.bufs[mid].bound_value >= 0) continue;
            bool other_use = false;
            for (size_t sj = 0; sj < plan.steps.size(); ++sj)
                if (sj != si && sj != si + 1)
                    for (int b : plan.steps[sj].slot) other_use |= (b == mid);
            const PoolParams &po = m.po;
            Epilogue e = g.epi;                 // wanted: [f32 bias] [relu] and nothing else
            finalize_epilogue(e);
            if (other_use || g.sh != 2 || g.sw != 2 || g.N != 64 || g.y_dtype != DT_BF16 || po.dtype != DT_BF16 || po.C != 64 ||
                po.KH != 3 || po.KW != 3 || po.sh != 2 || po.sw != 2 || po.ph != 1 || po.pw != 1 || po.H != g.OH || po.W != g.OW ||
                po.OH != (g.OH - 1) / 2 + 1 || po.OW != (g.OW - 1) / 2 + 1 || !e.simple || e.t_op >= 0 ||
                (e.has_bias && e.bias_dtype != DT_F32) || (e.rest_n != 0 && !e.relu_last) ||
                (uint64_t)po.N * po.OH * po.OW * 64 * 2 >= ((uint64_t)1 << 31))
                continue;
            // Two forms of the fused kernel.  One fetches its patches from the channel-first planes themselves: the frame
            // copy in front of this step (the step before, whose result only this step reads) then goes, and the weights
            // are packed for that kernel's contraction order instead.  The other reads the frame (exactly four K tiles).
            bool direct = false;
            if (si > 0 && !plan.opts.no_stem_direct) {
                const Step &pd = plan.steps[si - 1];
                const int wbuf = c.slot[SL_W];
                const int wv = wbuf >= 0 ? plan.bufs[wbuf].bound_value : -1;
                auto pk = wv >= 0 ? plan.packs.find(wv) : plan.packs.end();
                bool frame_private = pd.kind == S_STEM_PAD && pd.slot[SL_Y] == c.slot[SL_X];
                for (size_t sj = 0; frame_private && sj < plan.steps.size(); ++sj)
                    if (sj != si && sj != si - 1)
                        for (int b : plan.steps[sj].slot) frame_private &= (b != pd.slot[SL_Y]);
                direct = frame_private && pk != plan.packs.end() && pk->second.stem == 1 && consumers[wv].size() == 1 &&
                         stem_direct_ok(pd.t_C, pd.st_H, pd.st_W, pk->second.KH, pk->second.KW, pd.st_ph, pd.st_pw) &&
                         (uint64_t)pd.t_N * pd.t_C * pd.st_H * pd.st_W * 2 < ((uint64_t)1 << 31);
                if (direct) {
                    c.stem_direct = 1;
                    c.t_N = pd.t_N; c.t_C = pd.t_C; c.st_H = pd.st_H; c.st_W = pd.st_W; c.st_ph = pd.st_ph; c.st_pw = pd.st_pw;
                    c.stem_kh = pk->second.KH; c.stem_kw = pk->second.KW;
                    c.bytes += (double)plan.bufs[pd.slot[SL_X]].bytes - (double)plan.bufs[pd.slot[SL_Y]].bytes;
                    c.slot[SL_X] = pd.slot[SL_X];
                    PackSpec &ps = pk->second;
                    ps.stem = 2; ps.pw = pd.st_pw; ps.Kp = STEM_DIRECT_KP; ps.bytes = (size_t)ps.O * STEM_DIRECT_KP * 2;
                }
            }
            if (!direct && (g.K != 256 || g.Kp != 256 || g.KH != 4)) continue;
            c.kind = S_STEM_POOL;
            c.sp_N = po.N; c.sp_PH = po.OH; c.sp_PW = po.OW;
            c.slot[SL_Y] = m.slot[SL_Y];
            c.name += "+" + m.name;
            c.kernel = direct ? "igemm_conv2d_bf16_stem_maxpool_direct" : "igemm_conv2d_bf16_stem_maxpool";
            c.bytes = c.bytes - (double)plan.bufs[mid].bytes + (double)plan.bufs[m.slot[SL_Y]].bytes;
            plan.steps.erase(plan.steps.begin() + (long)si + 1);
            if (direct) {
                plan.steps.erase(plan.steps.begin() + (long)si - 1);
                --si;
            }
        }
    }

    // A contraction on the kernel of igemm_direct.hip, which stores through any strides: a 2x2 / stride 2 max-pool of its result
    // alone is taken over the finished values (same bits: max commutes with the rounding), and the change of layout that only
    // moves its result becomes the way it stores.
    void fuse_direct_store()
    {
        for (size_t si = 0; si + 1 < plan.steps.size(); ++si) {
            Step &c = plan.steps[si];
            if (c.kind != S_IGEMM || !c.il.direct) continue;
            Epilogue e = c.ig.epi;
            finalize_epilogue(e);
            bool elementwise_only = true;                       // no operand of the result's shape (it would have the result's layout)
            for (int i = 0; i < e.n_ops; ++i) elementwise_only &= epi_host_op(e, i) < E_ADD || epi_host_op(e, i) > E_RDIV;
            if (!elementwise_only) continue;
            while (si + 1 < plan.steps.size()) {
                const Step &m = plan.steps[si + 1];
                const int mid = c.slot[SL_Y];
                if (mid < 0 || m.slot[SL_X] != mid || plan.bufs[mid].bound_value >= 0) break;
                bool other_use = false;
                for (size_t sj = 0; sj < plan.steps.size(); ++sj)
                    if (sj != si && sj != si + 1)
                        for (int b : plan.steps[sj].slot) other_use |= (b == mid);
                if (other_use) break;
                IgemmParams &p = c.ig;
                const PoolParams &po = m.po;
                if (m.kind == S_MAXPOOL && !p.pool && e.simple && p.ys_c == 1 && po.KH == 2 && po.KW == 2 && po.sh == 2 && po.sw == 2 && po.ph == 0 && po.pw == 0 &&
                    po.H == p.OH && po.W == p.OW && po.C == p.N && po.dtype == p.y_dtype) {
                    p.pool = 1;
                    p.OH = po.OH; p.OW = po.OW; p.OHW = po.OH * po.OW;
                    p.M = 4 * po.N * p.OHW;                      // the last row and column of an odd image are not computed
                    p.ys_n = (int64_t)p.OHW * p.N;
                    make_fast_div((uint32_t)p.OHW, p.div_ohw_mul, p.div_ohw_sh);
                    make_fast_div((uint32_t)p.OW, p.div_ow_mul, p.div_ow_sh);
                    c.kernel += "_maxpool";
                } else if (m.kind == S_TO_NCHW && p.ys_c == 1 && p.ys_p == p.N && m.t_C == p.N && m.t_P == p.OHW) {      // (not of another view of one channel's pixels)
                    p.ys_n = (int64_t)p.N * p.OHW; p.ys_p = 1; p.ys_c = p.OHW;
                } else {
                    break;
                }
                c.bytes += (double)plan.bufs[m.slot[SL_Y]].bytes - (double)plan.bufs[mid].bytes;
                c.slot[SL_Y] = m.slot[SL_Y];
                c.name += "+" + m.name;
                plan.steps.erase(plan.steps.begin() + (long)si + 1);
            }
        }
    }

    // A result of the pixel-on-lane kernels that nothing but the change of layout into Shape order reads is stored in that order at once.
    // The two forms that only store rows of channels give way to their neighbours that can: 256x256 tiles (64x64x56x56 -> 256 1x1 85.0 -> 55.7 us,
    // 32x2048x14x14 -> 1024 67.0 -> 53.8) and K split over the waves, there below 512 channels (64x128x8x8 -> 512 16.9 -> 12.8, 8x256x28x28 -> 256
    // 19.4 -> 17.1; 512 channels, that split and the transposition against Shape order: 64x512x8x8 -> 512 28.0 and 29.7, with a residual
    // 29.0 and 28.7, 4x512x28x28 -> 512 25.3 and 25.9, with a residual 26.3 and 25.9).
    void fuse_planes_store()
    {
        if (plan.opts.no_shape_order || plan.lean) return;
        for (size_t si = 0; si < plan.steps.size(); ++si) {
            Step &c = plan.steps[si];
            if (c.kind != S_IGEMM || c.pair || c.chain || c.stem || !c.il.lp || c.il.ws || c.il.c64 || c.il.s2pair || c.il.anyact || (c.il.run > 1 && c.ig.C >= 512)) continue;
            IgemmParams p = c.ig;
            const int mid = c.slot[SL_Y];
            if (p.in_dtype != RL_BF16 || mid < 0 || plan.bufs[mid].bound_value >= 0 || p.ys_c != 1 || p.ys_p != p.N || p.ys_n != (int64_t)p.OHW * p.N) continue;
            size_t sj = 0;
            int users = 0;
            for (size_t k = 0; k < plan.steps.size(); ++k)
                if (k != si)
                    for (int b : plan.steps[k].slot)
                        if (b == mid) { ++users; sj = k; }
            if (users != 1 || sj < si || plan.steps[sj].kind != S_TO_NCHW || plan.steps[sj].slot[SL_X] != mid || plan.steps[sj].t_C != p.N || plan.steps[sj].t_P != p.OHW) continue;
            const int y = plan.steps[sj].slot[SL_Y];
            bool other_use = false;                          // the result is there earlier
            for (size_t k = 0; k < sj; ++k)
                for (int b : plan.steps[k].slot) other_use |= b == y;
            p.ys_n = (int64_t)p.N * p.OHW; p.ys_p = 1; p.ys_c = p.OHW;
            finalize_epilogue(p.epi);
            if (other_use || !p.epi.simple || !planes_ok(p)) continue;
            if (p.epi.t_op >= 0) {
                // the residual in the order the caller or a step before gave it, if its change of layout is all that stands between
                int &r = c.slot[SL_E0 + epi_host_arg(p.epi, p.epi.has_bias ? 1 : 0)];
                size_t sk = plan.steps.size();
                int readers = 0;
                for (size_t k = 0; k < plan.steps.size(); ++k)
                    for (int q = 0; q < SL_COUNT; ++q)
                        if (plan.steps[k].slot[q] == r) {
                            if (q == SL_Y) sk = k;
                            else ++readers;
                        }
                if (sk >= si || plan.steps[sk].kind != S_TO_NHWC || plan.steps[sk].pair || plan.steps[sk].t_C != p.N || plan.steps[sk].t_P != p.OHW || plan.bufs[r].bound_value >= 0) continue;
                Step &k = plan.steps[sk];
                r = k.slot[SL_X];
                if (readers == 1) {
                    k.slot[SL_X] = k.slot[SL_Y] = -1;
                    k.pair = 2;
                    k.bytes = 0;
                    k.kernel = "(read by the contraction as it is)";
                }
            }
            c.ig.ys_n = p.ys_n; c.ig.ys_p = p.ys_p; c.ig.ys_c = p.ys_c;
            c.il.planes = 1;
            if (c.il.run > 1) c.il.run = 1;
            if (c.il.big) { c.il.big = 0; c.kernel.replace(c.kernel.find("256x256"), 7, "256x128"); }
            c.kernel += "_shape_order";
            c.slot[SL_Y] = y;
            // the change of layout stays in the list, as one that launches nothing
            Step &m = plan.steps[sj];
            m.slot[SL_X] = -1;
            m.pair = 2;
            m.bytes = 0;
            m.kernel = "(stored by the contraction)";
        }
    }

    // Two consecutive contraction steps of which the second does not use the first one's result, and which run the
    // same variant of the pixel-on-lane kernel (a stage's stride-2 convolution and its 1x1 projection), share one
    // launch: each alone leaves a quarter of the CUs idle, and the projection's short tiles fit into that gap.
    void pair_contractions()
    {
        if (plan.opts.no_pair) return;
        for (size_t si = 0; si + 1 < plan.steps.size(); ++si) {
            Step &a = plan.steps[si];
            Step &b = plan.steps[si + 1];
            if (a.kind != S_IGEMM || b.kind != S_IGEMM || a.pair || b.pair || a.stem || b.stem) continue;
            // a 3x3 / stride 2 convolution and the 1x1 / stride 2 projection of the same tensor: one contraction, the
            // projection riding on the centre tap; any other two contractions of one kernel variant: one grid
            const bool fused = plan.opts.s2_pair && a.slot[SL_X] >= 0 && a.slot[SL_X] == b.slot[SL_X] && conv3x3s2_pair_ok(a.ig, a.il, b.ig, b.il);
            if (!fused && !igemm_lp_can_pair(a.ig, a.il, b.ig, b.il)) continue;
            const int ya = a.slot[SL_Y], yb = b.slot[SL_Y];
            if (ya < 0 || yb < 0 || ya == yb) continue;
            bool dep = false;
            for (int s : b.slot) dep |= (s == ya);          // b reads (or overwrites) a's result
            for (int s : a.slot) dep |= (s == yb);          // a reads what b writes
            if (dep) continue;
            a.pair = 1; b.pair = 2;
            if (fused) {
                a.il.s2pair = 1;
                a.kernel = "igemm_conv2d_bf16_3x3s2_pair";
                b.bytes -= (double)plan.bufs[b.slot[SL_X]].bytes;     // the shared input is read once
            }
            a.flops += b.flops; a.bytes += b.bytes;
            b.flops = 0; b.bytes = 0;
            a.name += " | " + b.name;
            b.kernel = "(launched with the step before)";
            ++si;
        }
    }

    // K slices of the contraction over rows where it shares its launch: alone it is cut until it fills the chip, here the other one
    // fills a part of it, and slices that end in one round with it cost less (32x64x28x28 -> 64 3x3 f32: 392 tiles beside 765 workgroups of
    // 85 slices 61 us the layer, beside 41 slices' 369 50).  In shader cycles: three workgroups share a CU, what is left over runs half of a workgroup's
    // time longer, and the adding launch as in plan_tn.
    void reslice_beside(const Step &ig, Step &tn)
    {
        TnParams &p = tn.tn;
        const int dt = tn.t_dtype, part = tn.slot[SL_PART];
        if (p.splits < 2 || part < 0) return;
        const int BK = 128 / (int)dtype_size(dt);
        const int64_t na = (int64_t)((ig.ig.M + 63) / 64) * ((ig.ig.N + 63) / 64) * std::max(ig.il.splits, 1), nka = ig.il.splits > 1 ? ig.ig.split_tiles : (ig.ig.K + BK - 1) / BK;
        const int64_t tiles = (int64_t)((p.M + 63) / 64) * ((p.N + 63) / 64), nk = (p.P + BK - 1) / BK;
        const double share = tile_cost(TILE_64x64, dt, 1 << 20) / (double)((1 << 20) / 256), alone = tile_cost(TILE_64x64, dt, 1);
        double best = 1e30;
        int splits = p.splits, tiles_each = p.split_tiles;
        for (int64_t sp = 2; sp <= p.splits; ++sp) {
            const int64_t per = (nk + sp - 1) / sp, w = na + tiles * sp;
            if ((nk + per - 1) / per != sp) continue;
            const double work = (double)(na * nka + tiles * nk);
            double t = share * std::max(work / 256.0, w <= 768 ? (double)((w + 255) / 256) * work / (double)w : work / 256.0 + 1.5 * (double)std::min(per, nka));
            const double longest = (double)std::max(per, nka);
            t = std::max(t, std::max(alone * longest, share * (double)std::min<int64_t>(3, (w + 255) / 256) * longest)) + 8.0 * sp * p.M * (double)p.N / 2200.0;
            if (t < best) { best = t; splits = (int)sp; tiles_each = (int)per; }
        }
        p.splits = splits; p.split_tiles = tiles_each;
        plan.bufs[part].bytes = (size_t)round_up((int64_t)splits * p.M * p.N * 4, 256);
    }

    // A layer's two gradients (a direct-load contraction and one over rows, on 64x64 tiles) in one launch, if nothing between them
    // but layout changes: the earlier one then waits until the other's operands are there too.
    void pair_gradients()
    {
        if (plan.opts.no_pair || plan.lean) return;
        auto moves_only = [](const Step &s) { return s.kind == S_TO_NHWC || s.kind == S_TO_NCHW || s.kind == S_PAD_NHWC || s.kind == S_PACK; };
        auto writes = [](const Step &s, int b) { return b >= 0 && (s.slot[SL_Y] == b || s.slot[SL_PART] == b); };
        auto touches = [](const Step &s, int b) {
            for (int q : s.slot)
                if (q == b) return true;
            return false;
        };
        // whether step b may run beside, or before, step a
        auto independent = [&](const Step &a, const Step &b) {
            for (int q : a.slot)
                if (q >= 0 && (writes(b, q) || (writes(a, q) && touches(b, q)))) return false;
            return true;
        };
        for (size_t si = 0; si < plan.steps.size(); ++si) {
            if ((plan.steps[si].kind != S_IGEMM && plan.steps[si].kind != S_TN) || plan.steps[si].pair) continue;
            size_t sj = si + 1;
            while (sj < plan.steps.size() && moves_only(plan.steps[sj]) && independent(plan.steps[si], plan.steps[sj])) ++sj;
            if (sj == plan.steps.size()) continue;
            const Step &a = plan.steps[si], &b = plan.steps[sj];
            if (a.kind + b.kind != S_IGEMM + S_TN || a.kind == b.kind || b.pair || !independent(a, b)) continue;
            const Step &ig = a.kind == S_IGEMM ? a : b, &tn = a.kind == S_TN ? a : b;
            if (ig.chain || ig.stem || !igemm_grads_ok(ig.ig, ig.il, tn.tn, tn.t_dtype, tn.tn_tile)) continue;
            std::rotate(plan.steps.begin() + (long)si, plan.steps.begin() + (long)si + 1, plan.steps.begin() + (long)sj);
            Step &first = plan.steps[sj - 1], &second = plan.steps[sj];
            reslice_beside(first.kind == S_IGEMM ? first : second, first.kind == S_TN ? first : second);
            first.pair = 3; second.pair = 2;
            first.flops += second.flops; first.bytes += second.bytes;
            second.flops = 0; second.bytes = 0;
            first.name += " | " + second.name;
            first.kernel += " | " + second.kernel;
            second.kernel = "(launched with the step before)";
            si = sj;
        }
    }

    // A 3x3 weight gradient that has a launch of its own takes the kernel that reads the three taps of a filter row from one copy of the
    // rows, where it is ahead.  Its cost in shader cycles beside that of the square tiles (plan_tn): a K tile of one workgroup, of which a CU
    // holds one, 600, to start and end 15500, and the same adding launch.  Of 20 layers of 16 to 64 images the nine it takes run at 0.86 to 0.97 of
    // their time, those it leaves would at 0.98 to 1.08 (64x512x14x14 -> 64 57.1 against 59.2 us, 64x192x14x14 -> 192 55.9 and 55.0).
    void run_weight_gradients()
    {
        if (plan.opts.tn_run < 0) return;
        for (size_t si = 0; si < plan.steps.size(); ++si) {
            Step &s = plan.steps[si];
            if (s.kind != S_TN || s.pair || !igemm_tn_run_ok(s.tn, s.t_dtype)) continue;
            TnParams &p = s.tn;
            const int64_t nk = ((int64_t)p.P + 63) / 64, tiles = (int64_t)((p.M + 63) / 64) * ((p.C + 63) / 64) * 3;
            double best = plan.opts.tn_run ? 1e30 : s.tn_cost;
            int splits = 0, per_best = 0;
            for (int64_t sp = 1; sp <= std::min<int64_t>(nk, plan.opts.tn_run > 1 ? plan.opts.tn_run : 512); ++sp) {
                const int64_t per = (nk + sp - 1) / sp;
                if ((nk + per - 1) / per != sp || (sp > 1 && sp * p.M * p.N >= (int64_t)1 << 27)) continue;
                if (sp > 1 && s.slot[SL_PART] < 0) break;                          // (one slice of the square tiles: the results alone fill the chip)
                const double cost = (double)((tiles * sp + 255) / 256) * ((double)per * 600.0 + 15500.0) + (sp > 1 ? 6500.0 + 8.0 * sp * p.M * (double)p.N / 2200.0 : 0.0);
                if (cost < best || (plan.opts.tn_run > 1 && sp > splits)) { best = cost; splits = (int)sp; per_best = (int)per; }
            }
            if (!splits) continue;
            p.splits = splits; p.split_tiles = per_best;
            if (s.slot[SL_PART] >= 0) plan.bufs[s.slot[SL_PART]].bytes = (size_t)round_up(splits > 1 ? (int64_t)splits * p.M * p.N * 4 : 256, 256);
            s.tn_tile = 0;
            s.kernel = std::string("igemm_conv2d_grad_w_bf16_64x64x3_rows_run") + (splits > 1 ? "_splitk" : "");
        }
    }

    // Two changes of layout that follow one another, neither of which touches what the other writes, in one launch: a layer's dy and x, a
    // convolution's input and its residual, one gradient's way out and the other operand's way in.
    void pair_moves()
    {
        if (plan.opts.no_pair || plan.lean) return;
        auto moves = [](const Step &s) { return s.kind == S_TO_NHWC || s.kind == S_TO_NCHW || s.kind == S_PAD_NHWC; };
        for (size_t si = 0; si + 1 < plan.steps.size(); ++si) {
            // a move behind a contraction that it has nothing to do with (x of a weight gradient behind the input gradient) comes before it,
            // and so beside the move that the contraction waits for (64x128x28x28 3x3 bf16, both gradients 61.2 -> 58.4 us)
            if (moves(plan.steps[si]) && !plan.steps[si].pair && plan.steps[si + 1].kind == S_IGEMM && !plan.steps[si + 1].pair && !plan.steps[si + 1].chain) {
                size_t sj = si + 2;
                while (sj < plan.steps.size() && moves(plan.steps[sj]) && plan.steps[sj].pair == 2) ++sj;      // (stored by the contraction)
                if (sj < plan.steps.size() && moves(plan.steps[sj]) && !plan.steps[sj].pair) {
                    // no step before it touches what it writes, or writes what it reads (a cell's result is its h or c)
                    const int *mv = plan.steps[sj].slot;
                    bool apart = true;
                    for (size_t k = si; k < sj; ++k) {
                        for (int q : plan.steps[k].slot) apart &= q < 0 || q != mv[SL_Y];
                        for (int q : {SL_Y, SL_COUT, SL_HOUT, SL_PART}) apart &= mv[SL_X] < 0 || plan.steps[k].slot[q] != mv[SL_X];
                    }
                    if (apart && moves_pair_ok(move_params(plan.steps[si]), move_params(plan.steps[sj])))
                        std::rotate(plan.steps.begin() + (long)si + 1, plan.steps.begin() + (long)sj, plan.steps.begin() + (long)sj + 1);
                }
            }
            Step &a = plan.steps[si], &b = plan.steps[si + 1];
            if (!moves(a) || !moves(b) || a.pair || b.pair || a.slot[SL_Y] == b.slot[SL_Y] || a.slot[SL_Y] == b.slot[SL_X] || a.slot[SL_X] == b.slot[SL_Y]) continue;
            if (!moves_pair_ok(move_params(a), move_params(b))) continue;
            a.pair = 1; b.pair = 2;
            plan.spent = true;                           // the second one's result is there a step earlier
            a.bytes += b.bytes;
            b.bytes = 0;
            a.name += " | " + b.name;
            a.kernel += " | " + b.kernel;
            b.kernel = "(launched with the step before)";
            ++si;
        }
    }

    // A dense contraction whose K is split over workgroups ends in a launch that adds the slices.  When its result feeds
    // nothing but a small dense layer right behind it (an MLP's output layer), that launch computes the small layer as
    // well, a row per workgroup, and the tensor between the two groups never leaves LDS: a launch fewer on graphs
    // whose time is the number of their launches.
    void chain_small_dense()
    {
        if (plan.opts.no_dense_chain) return;
        for (size_t si = 0; si + 1 < plan.steps.size(); ++si) {
            Step &a = plan.steps[si];
            Step &b = plan.steps[si + 1];
            if (a.kind != S_IGEMM || b.kind != S_IGEMM || a.pair || b.pair || a.chain || b.chain || a.stem || b.stem) continue;
            const IgemmParams &pa = a.ig, &pb = b.ig;
            if (a.il.splits < 2 || !a.il.avec || !a.il.dma || a.il.lp || a.il.gates || b.il.gates) continue;
            if (pa.OHW != 1 || pb.OHW != 1 || pa.KH * pa.KW != 1 || pb.KH * pb.KW != 1) continue;                       // two dense layers
            if (pa.ys_c != 1 || pa.ys_n != pa.N || pa.N > REDUCE_DENSE_MAX_N1 || pa.M > 65535) continue;
            if (pb.M != pa.M || pb.K != pa.N || pb.K1 != pb.K || pb.N > REDUCE_DENSE_MAX_N2 || pb.xs_c != 1 || pb.xs_n != pa.N) continue;
            if (b.slot[SL_X2] >= 0 || pb.in_dtype != pa.y_dtype || pb.w_frag) continue;                                // its weights in rows
            const int h = a.slot[SL_Y];
            if (h < 0 || plan.bufs[h].bound_value >= 0 || b.slot[SL_X] != h) continue;                               // the result is the plan's own
            bool other = false;                                                                                        // ... and nobody else's
            for (size_t sj = 0; sj < plan.steps.size(); ++sj)
                for (int q = 0; q < SL_COUNT; ++q)
                    if (plan.steps[sj].slot[q] == h && !((sj == si && q == SL_Y) || (sj == si + 1 && q == SL_X))) other = true;
            if (other) continue;
            a.chain = 1; b.chain = 2;
            b.slot[SL_PART] = -1;                       // the small layer's own K split, if it had one, is not used
            b.il.splits = 1; b.ig.splits = 0; b.ig.split_tiles = 0;
            a.kernel += "+dense";
            a.name += " > " + b.name;
            a.flops += b.flops; a.bytes += b.bytes - 2.0 * plan.bufs[h].bytes;      // the tensor between them is neither written nor read
            b.flops = 0; b.bytes = 0;
            b.kernel = "(launched with the step before)";
            ++si;
        }
    }

    // liveness-based first-fit packing of workspace buffers
    void assign_workspace()
    {
        for (size_t si = 0; si < plan.steps.size(); ++si)
            for (int b : plan.steps[si].slot)
                if (b >= 0) {
                    BufDesc &d = plan.bufs[b];
                    // the second step of a pair runs when the first is launched; so does a small layer on the adding launch before it, which writes
                    // rows of its result while others still read the partial sums
                    const int at = plan.steps[si].pair == 2 || plan.steps[si].chain == 2 ? (int)si - 1 : (int)si;
                    if (d.first < 0) d.first = at;
                    d.last = (int)si;
                }
        std::vector<int> ws;
        for (size_t b = 0; b < plan.bufs.size(); ++b)
            if (plan.bufs[b].bound_value < 0 && plan.bufs[b].first >= 0) ws.push_back((int)b);
        std::sort(ws.begin(), ws.end(), [&](int a, int b) { return plan.bufs[a].first < plan.bufs[b].first; });
        std::vector<int> placed;
        size_t total = 0;
        for (int b : ws) {
            BufDesc &d = plan.bufs[b];
            std::vector<std::pair<size_t, size_t>> busy;
            for (int q : placed) {
                const BufDesc &o = plan.bufs[q];
                if (o.last >= d.first && o.first <= d.last) busy.push_back({o.offset, o.offset + o.bytes});
            }
            std::sort(busy.begin(), busy.end());
            size_t off = 0;
            for (auto &iv : busy) {
                if (off + d.bytes <= iv.first) break;
                if (iv.second > off) off = iv.second;
            }
            d.offset = off;
            total = std::max(total, off + d.bytes);
            placed.push_back(b);
        }
        plan.workspace_bytes = total;
    }
};

}  // namespace

rl_status build_plan(const Graph &g, Plan &plan, std::string &msg)
{
    Planner pl(g, plan, msg);
    return pl.run();
}

std::string describe_plan(const Plan &p)
{
    std::ostringstream o;
    o << "{\"workspace_bytes\": " << p.workspace_bytes << ", \"steps\": [";
    for (size_t i = 0; i < p.steps.size(); ++i) {
        const Step &s = p.steps[i];
        o << (i ? ", " : "") << "{\"name\": \"" << s.name << "\", \"kernel\": \"" << s.kernel << "\", \"group\": " << s.group
          << ", \"flops\": " << (long long)s.flops << ", \"bytes\": " << (long long)s.bytes;
        if (s.kind == S_IGEMM)
            o << ", \"M\": " << s.ig.M << ", \"N\": " << s.ig.N << ", \"K\": " << s.ig.K << ", \"epilogue_ops\": " << s.ig.epi.n_ops
              << ", \"k_split_waves\": " << (s.il.run == 2 || (s.il.direct && s.il.direct_slices > 1) ? 1 : 0) << ", \"channel_tile_major\": " << s.ig.nmajor << ", \"shape_order\": " << s.il.planes << ", \"k_split_workgroups\": " << (s.il.splits > 1 ? s.il.splits : 1);
        if (s.kind == S_ELTWISE) o << ", \"n\": " << (long long)s.el.n << ", \"chain_ops\": " << s.el.epi.n_ops;
        o << "}";
    }
    // workspace buffers with the steps between which each one holds live data (first writer .. last reader)
    o << "], \"buffers\": [";
    bool firstb = true;
    for (size_t i = 0; i < p.bufs.size(); ++i) {
        const BufDesc &d = p.bufs[i];
        if (d.bound_value >= 0 || d.first < 0) continue;
        o << (firstb ? "" : ", ") << "{\"offset\": " << d.offset << ", \"bytes\": " << d.bytes << ", \"first\": " << d.first << ", \"last\": " << d.last
          << "}";
        firstb = false;
    }
    o << "], \"packed_params\": [";
    bool firstp = true;
    for (auto &kv : p.packs) {
        o << (firstp ? "" : ", ") << "{\"value\": " << kv.first << ", \"bytes\": " << kv.second.bytes << "}";
        firstp = false;
    }
    o << "]}";
    return o.str();
}

void finalize_epilogue(Epilogue &e)
{
    int s = 0;
    e.has_bias = 0; e.t_op = -1; e.bias_ptr = nullptr; e.t_ptr = nullptr; e.bias_dtype = 0; e.t_dtype = 0;
    if (s < e.n_ops && epi_host_op(e, s) == E_BIAS) {
        const int a = epi_host_arg(e, s);
        e.has_bias = 1; e.bias_ptr = e.ptr[a]; e.bias_dtype = epi_host_dtype(e, a); ++s;
    }
    if (s < e.n_ops && epi_host_op(e, s) >= E_ADD && epi_host_op(e, s) <= E_RDIV) {
        const int a = epi_host_arg(e, s);
        e.t_op = epi_host_op(e, s); e.t_ptr = e.ptr[a]; e.t_dtype = epi_host_dtype(e, a); ++s;
    }
    e.simple = 1;
    e.rest_n = 0;
    e.rest_ops = 0;
    for (; s < e.n_ops; ++s) {
        const int op = epi_host_op(e, s);
        if (op <= E_RDIV || e.rest_n >= 8) { e.simple = 0; break; }      // E_BIAS .. E_RDIV take operands
        e.rest_ops |= (uint64_t)op << (8 * e.rest_n);
        e.rest_n++;
    }
    e.relu_last = (e.simple && e.rest_n == 1 && e.rest_ops == (uint64_t)E_RELU) ? 1 : 0;
}

void make_fast_div(uint32_t d, uint32_t &mul, uint32_t &sh)
{
    mul = 0; sh = 0;
    if (d < 2) return;
    uint32_t l = 0;
    while (((uint64_t)1 << l) < d) ++l;                  // ceil(log2 d) >= 1
    const uint64_t pw = (uint64_t)1 << (31 + l);         // 2^31 <= pw / d < 2^32; exact quotients for n < 2^31
    mul = (uint32_t)((pw + d - 1) / d);
    sh = l - 1;
}

rl_status run_steps(const Plan &plan, void *const *ptrs, hipStream_t stream, std::string &msg, hipEvent_t *events)
{
    size_t si = 0;
    auto P = [&](const Step &s, int slot) -> void * { return s.slot[slot] >= 0 ? ptrs[s.slot[slot]] : nullptr; };
    auto params = [&](const Step &t) {
        IgemmParams p = t.ig;
        p.x = P(t, SL_X); p.x2 = P(t, SL_X2); p.w = P(t, SL_W); p.y = P(t, SL_Y);
        for (int i = 0; i < RL_EPI_MAX_PTRS; ++i) p.epi.ptr[i] = P(t, SL_E0 + i);
        finalize_epilogue(p.epi);
        p.c_in = (const float *)P(t, SL_CIN); p.c_out = (float *)P(t, SL_COUT); p.h_out = P(t, SL_HOUT);
        p.partial = (float *)P(t, SL_PART);
        return p;
    };
    auto tn_params = [&](const Step &t) {
        TnParams q = t.tn;
        q.a = P(t, SL_X); q.b = P(t, SL_X2); q.y = P(t, SL_Y); q.partial = (float *)P(t, SL_PART);
        return q;
    };
    auto move = [&](const Step &t) {
        MoveParams m = move_params(t);
        m.src = P(t, SL_X); m.dst = P(t, SL_Y);
        return m;
    };
    for (const Step &s : plan.steps) {
        hipError_t er = hipSuccess;
        if (events) er = hipEventRecord(events[si], stream);
        ++si;
        if (er == hipSuccess) switch (s.kind) {
        case S_IGEMM: {
            if (s.pair == 2 || s.chain == 2) break; // went out with the step before
            if (s.pair == 3) {
                er = launch_igemm_grads(params(s), s.il, tn_params(plan.steps[si]), s.ig.in_dtype, stream);
                break;
            }
            if (s.chain == 1) {
                const Step &t = plan.steps[si];     // si already counts this step: the next one
                IgemmParams pa = params(s), pb = params(t);
                pa.skip_reduce = 1;
                er = launch_igemm(pa, s.il, stream);
                if (er == hipSuccess) {
                    ReduceDenseParams r{};
                    r.partial = pa.partial; r.splits = pa.splits; r.M = pa.M; r.N1 = pa.N;
                    r.epi1 = pa.epi; r.hs_n = pa.ys_n; r.hs_c = pa.ys_c; r.h_dtype = pa.y_dtype;
                    r.w2 = pb.w; r.w_dtype = pb.in_dtype; r.N2 = pb.N; r.Kp2 = pb.Kp;
                    r.epi2 = pb.epi; r.y = pb.y; r.y_dtype = pb.y_dtype; r.ys_n = pb.ys_n; r.ys_c = pb.ys_c;
                    er = launch_reduce_dense(r, stream);
                }
            } else if (s.pair == 1) {
                const Step &t = plan.steps[si];     // si already counts this step: the next one
                er = s.il.s2pair ? launch_conv3x3s2_pair(params(s), s.il, params(t), t.il, stream)
                                 : launch_igemm_lp_pair(params(s), s.il, params(t), t.il, stream);
            } else {
                er = launch_igemm(params(s), s.il, stream);
            }
            break;
        }
        case S_ELTWISE: {
            EltwiseParams p = s.el;
            p.x = P(s, SL_X); p.y = P(s, SL_Y);
            for (int i = 0; i < RL_EPI_MAX_PTRS; ++i) p.epi.ptr[i] = P(s, SL_E0 + i);
            finalize_epilogue(p.epi);
            er = launch_eltwise(p, stream);
            break;
        }
        case S_GATES: {
            GatesParams p = s.ga;
            p.z = (const float *)P(s, SL_X); p.c_in = (const float *)P(s, SL_CIN); p.c_out = (float *)P(s, SL_COUT); p.h_out = P(s, SL_HOUT);
            er = launch_lstm_gates(p, stream);
            break;
        }
        case S_MAXPOOL: case S_GAVG: {
            PoolParams p = s.po;
            p.x = P(s, SL_X); p.y = P(s, SL_Y);
            er = s.kind == S_MAXPOOL ? launch_maxpool_nhwc(p, stream) : launch_gavgpool_nhwc(p, stream);
            break;
        }
        case S_TO_NHWC: case S_TO_NCHW: case S_PAD_NHWC:
            if (s.pair == 2) break;                 // went out with the step before
            er = s.pair == 1 ? launch_move_pair(move(s), move(plan.steps[si]), stream) : launch_move(move(s), stream);
            break;
        case S_STEM_POOL: {
            if (s.stem_direct) {
                StemDirectParams q{};
                q.x = P(s, SL_X); q.w = P(s, SL_W);
                q.x_bytes = (uint32_t)((uint64_t)s.t_N * s.t_C * s.st_H * s.st_W * 2);
                q.w_bytes = (uint32_t)(64 * STEM_DIRECT_KP * 2);
                q.epi = s.ig.epi;
                for (int i = 0; i < RL_EPI_MAX_PTRS; ++i) q.epi.ptr[i] = P(s, SL_E0 + i);
                finalize_epilogue(q.epi);
                q.yp = P(s, SL_Y);
                q.yp_bytes = (uint32_t)((uint64_t)s.sp_N * s.sp_PH * s.sp_PW * 64 * 2);
                q.n_img = s.sp_N; q.C = s.t_C; q.H = s.st_H; q.W = s.st_W; q.KH = s.stem_kh; q.KW = s.stem_kw; q.ph = s.st_ph; q.pw = s.st_pw;
                q.OH = s.ig.OH; q.OW = s.ig.OW; q.PH = s.sp_PH; q.PW = s.sp_PW;
                er = launch_stem_pool_direct(q, stream);
                break;
            }
            StemPoolParams q{};
            q.g = s.ig;
            q.g.x = P(s, SL_X); q.g.w = P(s, SL_W); q.g.y = nullptr;
            for (int i = 0; i < RL_EPI_MAX_PTRS; ++i) q.g.epi.ptr[i] = P(s, SL_E0 + i);
            finalize_epilogue(q.g.epi);
            q.yp = P(s, SL_Y);
            q.n_img = s.sp_N; q.PH = s.sp_PH; q.PW = s.sp_PW;
            q.kh = s.stem_kh;
            q.yp_bytes = (uint32_t)((uint64_t)s.sp_N * s.sp_PH * s.sp_PW * 64 * 2);
            er = launch_stem_pool(q, stream);
            break;
        }
        case S_PERMUTE: {
            PermuteParams p = s.pe;
            p.x = P(s, SL_X); p.y = P(s, SL_Y);
            er = launch_permute(p, stream);
            break;
        }
        case S_PACK:
            er = launch_pack_gather(P(s, SL_X), P(s, SL_Y), s.gp, stream);
            break;
        case S_WGRAD: {
            WgradParams q = s.wg;
            q.xT = P(s, SL_X); q.dyT = P(s, SL_X2); q.part = (float *)P(s, SL_PART);
            q.dy_bytes = (uint32_t)((uint64_t)q.OH * q.OW * q.O * 64 * q.nck * 2);
            q.x_bytes = (uint32_t)((uint64_t)q.H * q.W * q.C * 64 * q.nck * 2);
            er = launch_conv_wgrad(q, stream);
            break;
        }
        case S_TN:
            if (s.pair == 2) break;
            if (s.pair == 3) {
                const Step &t = plan.steps[si];     // si already counts this step: the next one
                er = launch_igemm_grads(params(t), t.il, tn_params(s), s.t_dtype, stream);
                break;
            }
            er = s.tn_tile ? launch_igemm_tn(tn_params(s), s.t_dtype, s.tn_tile, stream) : launch_igemm_tn_run(tn_params(s), s.t_dtype, stream);
            break;
        case S_DILATE:
            er = launch_dilate_nhwc(P(s, SL_X), P(s, SL_Y), s.t_N, s.st_H, s.st_W, s.st_Hp, s.st_Wp, s.t_C, s.st_ph, stream);
            break;
        case S_WGRAD_REDUCE:
            er = launch_wgrad_reduce((const float *)P(s, SL_X), P(s, SL_Y), s.t_dtype, s.t_N, s.t_C, s.wg.O, s.wg.C, stream);
            break;
        case S_STEM_PAD:
            er = launch_stem_pad(P(s, SL_X), P(s, SL_Y), s.t_N, s.t_C, s.st_H, s.st_W, s.st_Hp, s.st_Wp, s.st_ph, s.st_pw, stream);
            break;
        }
        if (er != hipSuccess) {
            msg = "launch of " + s.kernel + " (" + s.name + ") failed: " + hipGetErrorString(er);
            return RL_ERR_HIP;
        }
    }
    if (events && hipEventRecord(events[si], stream) != hipSuccess) { msg = "hipEventRecord failed"; return RL_ERR_HIP; }
    return RL_OK;
}

}  // namespace rl
