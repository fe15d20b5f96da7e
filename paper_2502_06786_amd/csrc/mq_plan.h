// How the calls of the linear layer and of the decode GEMV are cut into tiles, ranges and rounds: rules on sizes, host arithmetic
// without HIP.
//
// The constants of the linear layer and the times beside them were fitted to kernels on the 32x32x16 product.  With the 16x16x32 product the large
// sizes are 7-18 % faster and the choices are on average 2.4 / 2.7 / 1.8 % slower than the best (forward, 1 / 2 / 3 bit-widths; dX
// 0.8 / 1.2 % at one / three).  A refit of the forward gave 1.6 / 2.3 / 1.0 % and made 25 of 570 sizes 4-15 % slower: not taken.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace mq {

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

constexpr int BKT = 64;                  // contraction elements per LDS stage

// ============================================================================================
// forward
// ============================================================================================
constexpr int FWD_BN = 128;
constexpr int FWD_Q_TILE = FWD_BN * 64;
constexpr int FWD_STAGES = 4;

// 32-token blocks per workgroup of the tiled forward kernel: the accumulators (16 NR MB registers) must leave room for
// the operands
constexpr int fwd_mb(int nr) { return nr == 3 ? 5 : 6; }
constexpr double kFwdCycleNs = 0.47;  // ns per cycle of fwd_tiled_cost

// Token-tile height: the tallest tile amortises the code conversion and the epilogue best, but the
// number of tiles rarely divides evenly over the 256 compute units; one block less can save a whole
// round of workgroups.  Cost of a choice = rounds x (main loop + epilogue) in matrix-core cycles
// (32 per MFMA, plus about 180 cycles per 64-wide k stage and bit-width that do not shrink with the tile:
// conversions and the stage barrier - fitted on the 9B gate shape, where 160 tokens run 2.5-4 % faster than
// 128 although both fill their rounds; prologue and epilogue constants measured on the Gemma-2-2B shapes).
//
// Three bit-widths have the low tiles with two workgroups per compute unit as well, and a cost of their own, a fit to 640 timed
// combinations (8 layers of 2000 x 1008 to 14336 x 4096, 100 to 4096 tokens, plain and with the objective), in ns: a 64-wide
// stage takes 294 + 159 per token block, for two workgroups together 409 + 367 per block.  The choice, with the form that cuts
// K, is 0.6 % slower than the best of them on average, 13 % at worst (before: 6.5 %, 75 %).  r = 8/4/2 with the objective:
// 2000 x 1008, 700 tokens 35.8 -> 23.6 us; 3600 x 3600, 1400 tokens 140 -> 112 us; 12000 x 912, 2011 tokens 167 -> 145 us;
// 9216 x 2304, 2800 tokens 334 -> 311 us; the high tiles stay for 14336 x 4096, 2011 tokens (568 us).
//
// The result is the modelled cost (matrix-core cycles) at the best tile height, which goes to *mb unless null.
inline int64_t fwd_tiled_cost(int64_t M, int64_t N, int64_t K, int nr, int *mb) {
    const int hi = fwd_mb(nr);
    if (nr == 3) {
        const double stages = (double)cdiv(K, BKT);
        double best_ns = 0;
        for (int h = hi; h >= 2; --h) {
            const int64_t tiles = cdiv(M, 32 * h) * cdiv(N, FWD_BN), per_cu = cdiv(tiles, 256);
            if (tiles > 0x7FFFFFFF) continue;  // more than a launch takes (never at 128 tokens and more: fwd_run)
            const double ends = 871.0 + 1907.0 * h, alone = stages * (294.0 + 159.0 * h) + ends;
            const double ns = h > 3 ? per_cu * alone : per_cu / 2 * (stages * (409.0 + 367.0 * h) + 1.4 * ends) + per_cu % 2 * alone;
            if (h == hi || ns < best_ns) {
                best_ns = ns;
                if (mb) *mb = h;
            }
        }
        return (int64_t)(best_ns / kFwdCycleNs);
    }
    int64_t best = 0;
    for (int h = hi; h >= hi - 1; --h) {
        const int64_t tiles = cdiv(M, 32 * h) * cdiv(N, FWD_BN);
        const int64_t rounds = cdiv(tiles, 256);
        const int64_t per_tile = cdiv(K, BKT) * (nr * h * 128 + 180 * nr) + 3000 + 890 * nr * h;
        if (h == hi || rounds * per_tile < best) {
            best = rounds * per_tile;
            if (mb) *mb = h;
        }
    }
    return best;
}

// ---- one bit-width, 256-channel tiles (mq_linear_wide.hip) ------------------------------------
// The tiles are those of dX: DX_BK code rows, four waves of DX_RB blocks each.
constexpr int DX_MB = 5;                        // most 32-token blocks per wave
constexpr int DX_RB = 2;                        // 32-row blocks of k per wave
constexpr int DX_BK = 4 * 32 * DX_RB;           // k rows per workgroup (4 waves)
constexpr int DX_Q_TILE = DX_BK * 64;
// Row stride of the output staging tile: 16 bytes more than a row, so that the 8-byte writes of sixteen tokens spread over all banks
// and the read-back in pieces of 16 bytes stays aligned.
constexpr int DX_OS = DX_BK * 2 + 16;
static_assert(DX_OS % 16 == 0, "rows of the staging tile are read in aligned pieces of 16 bytes");
constexpr int dx_lds(int mb) {                  // four stages; the staging tile of the epilogue is smaller
    return 4 * (mb * 4096 + DX_Q_TILE);
}

// Which tile the forward at one bit-width takes where K is not split: rounds of workgroups times the time of a tile, in ns, a fit
// to 650 timed combinations (10 layers of 2000 x 1008 to 14336 x 4096, 100 to 4096 tokens).  Wide tiles are half as many, so
// they lose while the narrow ones still fit one round (3600 x 3600, 1000 tokens 45 against 54 us) and win from the second
// round on; with the form that cuts K the choice is 0.2 % slower than the best on average, 4 % at worst.  int4, narrow -> chosen: 14336 x 4096,
// 2011 tokens 256 -> 221 us, 4096 tokens 501 -> 425 us; 2304 x 9216, 4096 tokens 199 -> 168 us; 3600 x 3600, 1600 tokens 82
// -> 59 us; 2000 x 1008, 4096 tokens 34 -> 28.5 us.
// The result is the height of the better wide tile in blocks of 32 tokens, or 0 where the tiles of fwd_kernel are faster; *ns,
// unless null, the modelled time of the choice.
inline int fwd_wide_mb(int64_t M, int64_t N, int64_t K, double *ns) {
    double best = 0.678 * (double)fwd_tiled_cost(M, N, K, 1, nullptr);
    int choice = 0;
    for (int mb = 3; mb <= 6; ++mb) {
        const int64_t rounds = cdiv(cdiv(M, 32 * mb) * cdiv(N, DX_BK), 256);
        const double t = (double)rounds * ((double)cdiv(K, BKT) * (94.0 * mb + 402.0) + 3870.0 + 824.0 * mb);
        if (t < best) {
            best = t;
            choice = mb;
        }
    }
    if (ns) *ns = best;
    return choice;
}

// The losses of a forward with the objective: in grids of up to this many workgroups the last one to arrive finishes them (leave_sums),
// in larger ones a launch of one workgroup.  All workgroups add to one word, about 10 ns each; the launch takes 0.6 us between kernels and
// half a microsecond of the host.  Calls with the counter against calls with the launch at three bit-widths (2000 sizes each way; replayed
// from a graph, one after the other): 0.96 and 0.95 times as long up to 44 workgroups, 0.97 and 0.96 at 48 to 60.  At 128 (two rows of sums in a
// lane, 0.27 us more for everyone): 1.01 and 1.00 at 64 to 88, 1.03 and 1.02 at 92 to 124.  At 512 (sums added by all four waves): 1.04 and 1.02 at 128
// to 180, 1.10 at 256 to 360 and 1.13 at 364 to 504 in the form that cuts K, whole tiles 1.01.
constexpr int64_t kLossArrivals = 64;

// ---- few tokens: K split over workgroups (mq_linear_split.hip) --------------------------------
// most 32-token blocks per workgroup: at one bit-width two workgroups of three share a compute unit, one of four has it alone,
// and no size was found for which the rule below would take it
constexpr int split_mb(int nr) { return nr == 1 ? 3 : 4; }
constexpr int split_lds(int mb) { return FWD_STAGES * (mb * 32 * 128 + FWD_Q_TILE); }

// How the forward for few tokens cuts its work (mq_linear_split.hip); mb == 0: whole contractions are the better choice.
struct FwdSplitPlan {
    int mb, splits;       // 32-token blocks per workgroup, K ranges
    size_t part_bytes;    // fp32 accumulators of all ranges
    size_t rs_bytes;      // per-token sums of X per range
    int64_t loss_blocks;  // workgroups of the finishing kernel (rows of FwdArgs::partial)
};

// Which form, and how it is cut: the least modelled time in ns over one to four token blocks per workgroup and up to 16
// ranges of at least five 64-wide stages, against the tiled kernel.  Per stage a compute unit needs 128 cycles per
// matrix product row (32 x 64 x 32) and bit-width, 172 per bit-width for the conversions and 50 for the barrier, for each of
// the workgroups it holds (80 KB of LDS and 256 registers each where two fit), but never less than the 1000 cycles a stage
// takes to arrive; all workgroups together cannot read codes faster than 2900 or tiles of X faster than 4100 bytes per
// cycle; a workgroup starts and ends in 4200 cycles; launches and the finishing kernel cost 8500 cycles, 1800 bytes of
// accumulators take a cycle to be written and read back.  The constants are a fit; over 4770 timed combinations (10 layers of
// 256 x 256 to 36864 x 4608, 17 to 2000 tokens, one to three bit-widths) the choice is 1.7 % slower than the best cut that it
// weighs on average, 27 % at worst (2000 x 1008, 700 tokens, two bit-widths).  One range at more than 64 tokens is not
// weighed: it would pay on the smallest layers only (256 x 256, 77 to 700 tokens 9.3 us against 12.5).  Measured, tiled ->
// chosen: 4096 x 4096, 77 tokens, int4 38.7 -> 17.8 us; 4096 x 14336 115 -> 26 us; 2304 x 9216 at r = 8/4/2, 203 tokens 86 ->
// 44 us; level with the tiled kernel at 700 (14336 rows: 200) tokens and more.
//
// The objective does not enter the rule, although its calls have no wide tiles to fall back on: the sums of a call with the
// objective have to run in the order of those of the call without.  It costs the former 4 % (at most 11 %) on the one size in
// 450 of 896 .. 14336 squared and 17 .. 2048 tokens, at one bit-width, where the wide tiles beat the cut (by 8 %).
inline FwdSplitPlan make_split_plan(int64_t M, int64_t N, int64_t K, int nr) {
    FwdSplitPlan best{0, 0, 0, 0, 0};
    if (M < 1 || N < 1 || M > 2048) return best;
    const int64_t tiles_n = cdiv(N, FWD_BN), nkt = cdiv(K, BKT);
    // with its row-sum pre-pass (for three bit-widths less the margin by which the fits of the two forms are apart)
    double best_cost = kFwdCycleNs * (double)fwd_tiled_cost(M, N, K, nr, nullptr) + (nr == 3 ? (double)M * K / 2000.0 - 500.0 : 4600.0);
    double wide;
    if (nr == 1 && fwd_wide_mb(M, N, K, &wide)) best_cost = std::min(best_cost, wide + 4600.0);
    for (int mb = 1; mb <= split_mb(nr); ++mb) {
        const int64_t tiles_m = cdiv(M, 32 * mb), tiles = tiles_m * tiles_n;
        if (mb > 1 && tiles_m == cdiv(M, 32 * (mb - 1))) continue;
        const int resident = std::max(1, std::min(163840 / split_lds(mb), 512 / (16 * nr * mb + 110)));
        const double busy = nr * mb * 128.0 + 172.0 * nr + 50.0;
        for (int splits = 1; splits <= 16; ++splits) {
            const int64_t stages = cdiv(nkt, splits);
            if (splits > 1 && stages < 5) break;
            if (splits == 1 && M > 64) continue;
            const size_t part = (size_t)splits * tiles * nr * mb * 16384;
            if (part > ((size_t)96 << 20)) break;
            const int64_t per_cu = cdiv(tiles * splits, 256), full = per_cu / resident, rest = per_cu % resident;
            double loop = full * std::max(resident * busy, 1000.0) + (rest ? std::max(rest * busy, 1000.0) : 0.0);
            loop = loop * stages + (full + (rest ? 1 : 0)) * 4200.0;
            loop = std::max(loop, std::max((double)N * K / 2900.0, (double)tiles * splits * stages * mb * 4096.0 / 4100.0));
            const double cost = 0.51 * (loop + 8500.0 + part / 1800.0 + 217.0 * splits * nr);
            if (cost < best_cost) {
                best_cost = cost;
                best.mb = mb;
                best.splits = splits;
                best.part_bytes = part;
                best.rs_bytes = (size_t)splits * tiles_m * 32 * mb * 4;
                best.loss_blocks = tiles * mb * 4;
            }
        }
    }
    return best;
}

// ============================================================================================
// backward dX (mq_linear_wide.hip)
// ============================================================================================
// How dX cuts its work; splits == 1: no partial sums.
struct DxPlan {
    int mb, splits;     // 32-token blocks per workgroup, ranges of n
    size_t part_bytes;  // fp32 accumulators of all ranges
};

// Tile height and ranges: the least modelled time (cycles) over one to five token blocks per workgroup and up to 16 ranges of
// n.  160 tokens x 256 k tiles alone leave most compute units idle up to about 2000 tokens (16 tokens through 9216 x 2304 are
// nine workgroups that walk 432 stages each: 263 us), and a full partial round of low tiles often beats the same round of
// high ones.  A stage (one n tile, one bit-width) takes 256 cycles per token block for its products and 520 for conversions
// and the barrier, for each of the workgroups that a compute unit holds (two where the stages of 32 tokens fit twice into its
// LDS), but never less than the 1055 + 140 per token block it takes to arrive; all workgroups together do not get gradients
// faster than 3650 or codes faster than 6480 bytes per cycle; a tile's epilogue costs 900 per token block, the finishing
// launch 4100 and 310 per range, and 1940 bytes of accumulators go out and come back per cycle.  The constants are a fit; over
// 3500 timed combinations (8 layers of 256 x 256 to 14336 x 4096, 16 to 4096 tokens, one and three bit-widths) the choice
// is 0.7 % slower than the best of them on average, 18 % at worst (256 x 256, 2000 tokens, r = 8/4/2).  dX with its preparation, 160-token tiles -> chosen, at
// r = 8/4/2: 9216 x 2304, 16 tokens 263 -> 54 us, 400 tokens 342 -> 96 us, 2000 tokens 371 -> 274 us; 3600 x 3600, 400
// tokens 160 -> 73 us, 4096 tokens 388 -> 354 us; 256 x 256, 16 tokens 15.6 (32-token tile) -> 13.9 us; the same at
// 4096 tokens through 9216 x 2304 (499 us).
inline DxPlan make_dx_plan(int64_t M, int64_t N, int64_t K, int nr) {
    DxPlan best{DX_MB, 1, 0};
    double best_cost = 0;
    const int64_t tiles_k = cdiv(K, DX_BK), nnt = cdiv(N, BKT);
    for (int mb = DX_MB; mb >= 1; --mb) {
        const int64_t tiles = cdiv(M, 32 * mb) * tiles_k;
        if (mb > 1 && cdiv(M, 32 * mb) == cdiv(M, 32 * (mb - 1))) continue;  // a lower tile covers as much
        const int resident = 2 * dx_lds(mb) <= 163840 ? 2 : 1;
        const double busy = mb * 256.0 + 520.0, arrive = mb * 140.0 + 1055.0;
        for (int splits = 1; splits <= std::min<int64_t>(16, nnt); ++splits) {
            const size_t part = splits > 1 ? (size_t)splits * tiles * mb * DX_RB * 16384 : 0;
            if (splits > 1 && (part > ((size_t)96 << 20) || tiles * splits > 1100)) break;
            const int64_t per_cu = cdiv(tiles * splits, 256), full = per_cu / resident, rest = per_cu % resident;
            const int64_t n_stages = cdiv(nnt, splits), stages = n_stages * nr;
            double cost = full * std::max(resident * busy, arrive) + (rest ? std::max(rest * busy, arrive) : 0.0);
            cost = cost * stages + per_cu * mb * 900.0;
            cost = std::max(cost, (double)tiles * splits * (stages * mb * (4096.0 / 3650.0) + n_stages * (16384.0 / 6480.0)));
            if (splits > 1) cost += 4100.0 + 310.0 * splits + part / 1940.0;
            if (best_cost == 0 || cost < best_cost) {
                best_cost = cost;
                best = DxPlan{mb, splits, part};
            }
        }
    }
    return best;
}

// ============================================================================================
// backward dW (mq_linear.hip)
// ============================================================================================
constexpr int DW_BM = 32;                            // contraction elements (tokens) per stage: 64-byte rows
constexpr int DW_NST = 5;                            // LDS stages
constexpr int dw_side(int hb) { return 64 * hb; }    // rows of n and columns of k per workgroup: 2 x 2 waves of hb 32-blocks
constexpr int dw_lds(int hb) { return DW_NST * 2 * dw_side(hb) * 64; }
constexpr int DW_CUS = 256;                          // compute units a round of workgroups fills

// How the tiles of dW (of `batch` gradients together) are dealt to workgroups.  Two sizes of tile: 256 x 256 (hb = 4) has the
// smaller operand traffic per product, 128 x 128 (hb = 2) four times as many tiles, two of which fit a compute unit.  Whole
// rounds of 256 x 256 tiles run one tile per workgroup; the tiles of a last partial round (at most half a round) are cut
// along the tokens into `parts` ranges each, so that the round still occupies every compute unit for 1 / parts of a tile's
// time.  Where the tiles do not fill one round all of them may be cut.  The ranges leave fp32 partial tiles in the workspace
// and dw_reduce_kernel adds them in a fixed order.
//
// The choice is the least modelled time (cycles): a 32-token stage takes 1045 per 256-tile; of 128-tiles, 742 for two on a
// compute unit, 437 for one; a tile ends in 10700 (2100); a cut costs 1300, 2230 per range and a cycle per 4780 bytes of
// partial tiles written and read back.  The constants are a fit to 900 timed combinations (10 layers of 256 x 256 to
// 14336 x 4096, 16 to 8192 tokens); the choice is 0.3 % slower than the best of them on average, 10 % at worst.  dW with its
// preparation, 256-tiles -> chosen: 256 x 256, 16 tokens 12.5 -> 8.7 us, 4096 tokens 84 -> 24 us; 2000 x 1008, 400 tokens 23
// -> 14 us; 2304 x 2304, 2000 tokens 60 -> 45 us; 6400 x 1104, 4096 tokens 117 -> 93 us; 2304 x 9216, 1200 tokens 90 -> 80 us,
// 4096 tokens the same (201 us).
struct DwPlan {
    int hb, tiles_n, tiles_k, whole, rest, parts;
    size_t part_bytes;
};
inline DwPlan make_dw_plan(int64_t M, int64_t N, int64_t K, int batch) {
    DwPlan best{};
    double best_cost = 0;
    const int64_t stages = cdiv(M, DW_BM);
    const int64_t max_parts = std::max<int64_t>(1, stages / 8);  // at least eight stages per range
    for (int hb = 4; hb >= 2; hb -= 2) {
        const int side = dw_side(hb);
        const int64_t tiles_n = cdiv(N, side), tiles_k = cdiv(K, side), tiles = tiles_n * tiles_k * batch;
        auto rounds = [&](int64_t items, int64_t st) {
            const int64_t per_cu = cdiv(items, DW_CUS);
            if (hb == 4) return per_cu * (1045.0 * st + 10700.0);
            return (per_cu / 2 * 742.0 + per_cu % 2 * 437.0) * st + per_cu * 2100.0;
        };
        auto consider = [&](int64_t rest, int64_t parts) {
            const size_t bytes = (size_t)rest * parts * side * side * 4;
            double cost = rounds(tiles - rest, stages);
            if (rest > 0) cost += rounds(rest * parts, cdiv(stages, parts)) + 1300.0 + 2230.0 * parts + 2.0 * bytes / 4780.0;
            if (best_cost == 0 || cost < best_cost) {
                best_cost = cost;
                best = DwPlan{hb, (int)tiles_n, (int)tiles_k, (int)(tiles - rest), (int)rest, (int)parts, bytes};
            }
        };
        const int64_t over = tiles % DW_CUS;
        if (tiles < DW_CUS) {
            for (int64_t parts = 2; parts <= std::min<int64_t>(8, max_parts); ++parts)
                if ((size_t)tiles * parts * side * side * 4 <= ((size_t)96 << 20)) consider(tiles, parts);
        } else if (hb == 4 && over > 0) {
            const int64_t parts = std::min<int64_t>(DW_CUS / over, max_parts);
            if (parts >= 2) consider(over, parts);
        }
        // a last partial round of 256-tiles that can be cut is cut: whole tiles there cost a full round
        if (!(hb == 4 && best.rest > 0 && best.whole > 0)) consider(0, 1);
    }
    return best;
}

// The cut that needs no workspace.
inline DwPlan dw_plan_whole(int64_t N, int64_t K, int batch) {
    const int tiles_n = (int)cdiv(N, dw_side(4)), tiles_k = (int)cdiv(K, dw_side(4));
    return DwPlan{4, tiles_n, tiles_k, tiles_n * tiles_k * batch, 0, 1, 0};
}

// Whether dW takes its operands by rows of tokens and lets the LDS turn them (dw_kernel's TURN), or transposed copies that a preparation
// makes of them.  The copies are 4 bytes per element of X, and of the gradients if they could be taken as they stand (alone: not scaled or
// summed), written and read back at 5.1 TB/s.  Without them the kernel reads the LDS twice as often and rows far apart in memory:
// 10 to 20 % longer on 256-tiles (18432 x 2304, 4096 tokens 286 -> 314 us, 2304 x 9216, 1999 tokens 231 -> 256), 30 to 70 % on
// 128-tiles (hb = 2), up to 40 % where a row by itself is no multiple of the 128 bytes of a line (3600 x 1808, 700 tokens, three
// gradients 36 -> 49); of 2 M N K flops a gradient at 1.4 PFLOP/s.  The preparation is a launch of its own, 4 us, unless it runs anyhow (prep:
// operands of dX, a summed or scaled gradient); beside its other work the copies cost less than their bytes.
//
// Whole calls at 1671 pairs of times (700 sizes of 512 to 14336 rows and columns, 90 to 8192 tokens; backward with and without dX, clip
// gradients): where operands are taken as they stand a call is 0.887 times as long on average, longer by more than 0.5 % at three
// sizes (2034 tokens through 2560 x 4096 103.6 -> 105.4 us).  128-tiles with a preparation were up to 13 % slower in a backward (59 of 100
// sizes by more than 1 %), 19 % without dX (2816 x 1408, 8192 tokens, one scaled gradient 85 -> 99 us).
// Few tokens make small copies: 4960 x 3712, 229 tokens 21 -> 23.5 us, preparation the same; the block of 1392 and 1408 columns, 886
// tokens (copies of 10 MB) 254 -> 261 us a call.  (A single gradient without dX would gain below these limits too.)
inline bool dw_turns(int64_t M, int64_t N, int64_t K, int batch, bool alone, bool prep, int hb) {
    const double columns = (double)K + (alone ? (double)batch * N : 0.0);
    if (M < 768 || (double)M * columns * 4.0 < 16.0 * 1048576.0) return false;
    const double copies = columns * 4.0 / 5.1e6, products = 2.0 * batch * (double)N * K / 1.4e9;   // us per token
    if (hb == 2) return !prep && M * copies + 4.0 > 0.7 * M * products;
    const bool lines = K % 64 == 0 && (!alone || N % 64 == 0);
    return copies > (!lines ? 0.4 : prep ? 0.22 : 0.13) * products;
}

// Whether two pieces of memory share a byte.
inline bool bytes_meet(const void *a, size_t a_bytes, const void *b, size_t b_bytes) {
    const uintptr_t pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
    return pa < pb + b_bytes && pb < pa + a_bytes;
}

// The same for a backward, whose outputs may lie over its inputs: X, and the gradient if it is the operand as it stands (dY; otherwise null),
// are then copied first.  dX is stored before dW is formed, and workgroups of dW still read their operands while others store.
inline bool dw_turns_in_place(int64_t M, int64_t N, int64_t K, const void *X, const void *dY, const void *dX, const void *dW, bool prep, int hb) {
    const size_t x_bytes = (size_t)M * K * 2, dw_bytes = (size_t)N * K * 4;
    auto stored_over = [&](const void *in, size_t bytes) { return bytes_meet(dW, dw_bytes, in, bytes) || (dX && bytes_meet(dX, x_bytes, in, bytes)); };
    if (stored_over(X, x_bytes) || (dY && stored_over(dY, (size_t)M * N * 2))) return false;
    return dw_turns(M, N, K, 1, dY != nullptr, prep, hb);
}

// Whether a backward forms dW before dX.  Each comes soonest right after the launch that has written its operands, while they are in the
// caches.  dX is the general choice: the fp32 dW in between pushes the codes and scaled gradients out (dW first, 4-bit, 270 tokens, 6576 x 11376
// 197.8 -> 218.8 us).  Where all of dW's share is about the size of the L2s and its operands are not small beside it, it goes first (r = 8/4/2,
// 687 tokens, 816 x 1952 39.3 -> 37.3 us).  4200 pairs of times with either order: 0.997 times as long as with dX first always
// (0.906 to 1.058), 0.996 as with dW first always (0.861 to 1.044; 349 of 2118 against 120 longer by more than 1 % than with the better order).
inline bool dw_first(int64_t M, int64_t N, int64_t K) {
    const double operands = 2e-6 * (double)M * (double)(N + K), out = 4e-6 * (double)N * K;   // MB
    return operands + out <= 48.0 && operands >= 2.0 + 0.1 * out;
}

constexpr int GEMV_TILE = 2048;                  // decode: 16 rows x one 128-byte line

// ============================================================================================
// decode GEMV for up to four sequences on tall planes (mq_gemv_quad.hip)
// ============================================================================================
constexpr int QUAD_SUM_BYTES = 1024;
constexpr int QUAD_X_PAD = 32;

// Waves of a workgroup that walk the list, next to nw that stream the plane: four or eight in all, because a workgroup's waves are
// dealt to the four SIMDs from the first one on (three workgroups of 3 + 2 waves do not share a compute unit), and at least one per
// streaming wave.  36864 x 4608 int2, 5 % of the entries: 3 + 5 waves take 20.8 / 22.4 / 24.9 us at B = 1 / 2 / 4, 3 + 1 waves
// 29.6 / 32.3 / 53.2, a launch of its own for the list 26.4 / 27.7 / 30.9.
constexpr int quad_list_waves(int nw) { return nw < 3 ? 4 - nw : 8 - nw; }

// With four waves for the list and three or four sequences the list of a dense matrix outlasts the plane: there the waves that
// stream the plane take rows of the list as well when they are done.  28672 x 4096, B = 4: at 12.5 % of the entries (uniform codes
// at int2) 30.5 -> 27.6 us, int4 31.4 -> 29.6 (a launch of its own for the list 27.9 and 30.0), at 5 % 19.6 -> 18.5 and 20.6 -> 20.8,
// at 2 % 16.3 -> 16.6 and 17.4 -> 18.1; 16384 x 4096, two row blocks per workgroup, all of whose rows are taken by then, 13.5
// and 19.2 us at 5 and 12.5 % either way (15.6 and 18.9).  Elsewhere the counter costs more than it gives: 16384 x 1024, B = 2 8.2
// -> 8.9 us.
constexpr bool quad_list_shared(int nw, int64_t B) { return nw == 4 && B >= 3; }

struct QuadPlan {
    int nl, nsl, ks, rw, ch, grid;
    int depth;                 // tiles in a wave's ring; 0: the form is not used
    int list_waves;            // 0: without a list
    bool shared;               // quad_list_shared
    size_t lds;
};
inline QuadPlan make_quad_plan(int64_t B, int64_t N, int64_t K, int64_t KB, int r, bool list) {
    QuadPlan p{};
    if (B > 4 || (r != 2 && r != 4)) return p;
    const int lines = (int)cdiv(KB, 128);
    const int nrb = (int)cdiv(N, 16);
    // Measured against the general kernel on 4096..36864 rows: 0.85-0.9x the time at 36864 x 4608, level or
    // slower at 14336 rows and below, where a launch is bound by latencies and not by bytes.
    if (nrb < 1024) return p;
    // Lines per slice: no padded lines if possible, then about four slices per row (measured over the
    // decode shapes: fewer leave a workgroup with too few waves, more spend their time filling activation
    // registers), one round.
    {
        int best = -1, best_cost = 0;
        for (int nl = 1; nl <= 4; ++nl) {
            const int nsl = (lines + nl - 1) / nl, pad = nsl * nl - lines;
            const int cost = pad * 8 + (nsl > 8 ? 4 : 0) + (nsl > 4 ? nsl - 4 : 4 - nsl);
            if (best < 0 || cost < best_cost) best = nl, best_cost = cost;
        }
        p.nl = best;
    }
    p.nsl = (lines + p.nl - 1) / p.nl;
    // Slices per round: all of them up to eight waves, otherwise the largest divisor (every wave the
    // same number of rounds), otherwise eight.
    p.ks = std::min(p.nsl, 8);
    if (p.nsl > 8)
        for (int d = 8; d >= 5; --d)
            if (p.nsl % d == 0) {
                p.ks = d;
                break;
            }
    // With the list only where at least as many waves are left for it.  Launch of its own -> here, 5 % of the entries unless noted:
    // 16384 x 1024, B = 2 10.3 -> 8.3 us; 20000 x 2048, B = 3 16.1 -> 12.3; 28672 x 8192, B = 2 30.5 -> 25.6; 73728 x 4608, B = 1
    // 37.5 -> 28.7; int4 28672 x 4096, B = 4 24.4 -> 20.8; 36864 x 4608 at 12.5 %, B = 4 38.5 -> 33.9.  Five to
    // seven streaming waves: level at 5, 32.8 -> 27.9 us or 47.3 -> 67.4 (2 and 12.5 % of the entries) at 6, 18.9 -> 35.1 at 7.
    // (Lists denser than those of uniform codes are faster in a launch of their own, by 3-15 % at 25 % of the entries from B = 2 on;
    // the host knows how much a list can hold and not how much it does.)
    if (list && quad_list_waves(p.ks) < p.ks) return p;
    // waves per compute unit the grid is sized for (measured on 16384..73728 rows: 12 is best at B = 1, within 2 % of the
    // best everywhere; at B = 4, where a wave's activation registers take four times as long to fill, 8 is 5-10 % faster
    // on the tall planes; 6, 16 and 24 are slower)
    const int wpc = B > 2 ? 8 : 12;
    // Row-block waves per workgroup and row blocks per workgroup: the whole grid resident at once
    // (wpc waves per compute unit), every wave the same number of visits where the shape allows.
    p.rw = 1;
    const int nw = p.ks * p.rw;
    int per_cu = std::max(1, wpc / nw);
    if (list) {
        p.list_waves = quad_list_waves(nw);
        p.shared = quad_list_shared(nw, B);
        per_cu = std::min(per_cu, 16 / (nw + p.list_waves));  // (128 registers: sixteen waves to a compute unit)
    }
    const int capacity = 256 * per_cu;
    const int visits = (int)cdiv(nrb, (int64_t)capacity * p.rw);  // per wave and round
    p.ch = visits * p.rw;
    p.grid = (int)cdiv(nrb, p.ch);
    p.ch = (int)cdiv(nrb, p.grid);  // (the most row blocks any workgroup gets)
    // Ring depth, as far as the LDS of a compute unit (160 KB, shared by per_cu workgroups) allows.
    const size_t fixed = QUAD_SUM_BYTES + (size_t)p.nsl * p.ch * 256 + (size_t)B * (((size_t)K + 511) / 512 * 1024 + QUAD_X_PAD) +
                         (list ? (size_t)p.ch * 16 * 24 + 16 : 0);
    const size_t budget = (size_t)160 * 1024 / per_cu;
    if (N * KB > 0x7FFFFFFFll || B * K * 2 > 0x7FFFFFFFll) return p;
    for (int d : {3, 2}) {  // (deeper rings measured slower: three steps in flight per wave are enough)
        p.lds = fixed + (size_t)nw * d * GEMV_TILE;
        if (p.lds <= budget) {
            p.depth = d;
            break;
        }
    }
    return p;
}

// ============================================================================================
// decode GEMV, general form (mq_gemv.hip)
// ============================================================================================
constexpr int line_bytes(int r) { return (r == 6 || r == 3) ? 96 : 128; }  // what eight neighbouring lanes fetch of a row
constexpr int line_codes(int r) { return line_bytes(r) * 8 / r; }          // k values per line
constexpr int GEMV_SUM_BYTES = 1024;

// The kernel has two row groups per wave (rg) at most.  These forms take more than 128 registers if they may: 147 and 131 at int2
// and int6 with two row groups, 134 and 156 at int3 with one and two.  Held to 128 they spill inside the main loop (14336 x 4096
// int2, B = 4: 9.8 us instead of 8.75), but two workgroups of eight waves fit a compute unit.
constexpr bool gemv_roomy(int r, int rg) { return r == 3 || (rg == 2 && (r == 2 || r == 6)); }

struct GemvPlan {
    int rg, ks, nw;           // 16-row groups per wave, waves that share a row block along K, waves of a workgroup
    int blocks, single;       // 512-k blocks of x staged at a time; all of x at once
    int ngroups, grid;        // groups of row blocks a workgroup takes at a time, workgroups
    bool tight;               // held to 128 registers (forms that are gemv_roomy)
    size_t x_off, lds;
};
inline GemvPlan make_gemv_plan(int64_t B, int64_t N, int64_t KB, int r) {
    GemvPlan p{};
    // Rows per wave (16 RG): every activation operand read from LDS serves RG matrix-core products, so
    // tall matrices take two row groups; short ones keep RG = 1 for more waves (measured on the decode
    // shapes at B = 4 and 16: 4096 rows run 10-25 % faster with RG = 1, 14336 rows level or faster with 2;
    // at B = 1 the columns are idle anyway and 11008 and 14336 rows run 6-13 % faster with RG = 1.  A
    // deeper ring did not help at any of these sizes: D = 4 and 5 were 2-10 % slower than 3).
    p.rg = (N >= 8192 && (B > 2 || N >= 16384)) ? 2 : 1;
    // K-split: about 2048 waves in total (8 per compute unit measured best across the decode shapes:
    // enough loads in flight, and the whole grid resident at once) when there are few row blocks,
    // none when the rows alone provide them.  Workgroups have 8 waves (KS of them per row block),
    // or KS when that is larger.
    const int64_t lines = cdiv(KB, line_bytes(r));  // weight lines per row
    const int64_t row_blocks = cdiv(N, 16 * p.rg);
    p.ks = 1;
    // (short matrices with batched activations: shorter slices pay off; at 14336 rows they cost 15-25 %)
    const int64_t wave_budget = (B >= 4 && p.rg == 1) ? 4096 : 2048;
    while (p.ks < 16 && row_blocks * p.ks * 2 <= wave_budget && 2 * p.ks <= lines) p.ks <<= 1;
    p.nw = p.ks > 8 ? p.ks : 8;

    int bp = 1;
    while (bp < B) bp <<= 1;
    const int SSPB = 512 / line_codes(r);             // weight lines per 512-k block of x
    const int blocks_all = (int)cdiv(lines, SSPB);    // 512-k blocks that cover K
    // area A: the 2 KB transposition tiles of the waves (reused for the K-split partial sums, which
    // need RG <= 2 KB per wave)
    constexpr size_t kLds = 160 * 1024;
    // all of x at once when it fits behind the reduction data; otherwise chunks that are a multiple of
    // KS * D lines, so that the register ring of every wave is in the same phase at each chunk
    // boundary, restaged for every group of row blocks, with the reduction data laid over them
    p.blocks = blocks_all;
    p.single = 1;
    p.x_off = (size_t)p.nw * 2048;
    p.lds = GEMV_SUM_BYTES + p.x_off + (size_t)blocks_all * bp * 1024;
    if (p.lds > kLds) {
        p.single = 0;
        // chunks of whole 512-k blocks whose line count is a multiple of KS; eight waves per workgroup
        // (more row-block groups, a smaller area A), the largest KS whose chunk still fits (at KS = 1 at least seven 16 KB blocks)
        p.nw = 8;
        if (p.ks > p.nw) p.ks = p.nw;
        p.x_off = (size_t)p.nw * 2048;
        int cap_blocks = 0;
        for (;; p.ks >>= 1) {
            cap_blocks = (int)(std::min<size_t>(131072, kLds - GEMV_SUM_BYTES - p.x_off) / (bp * 1024));
            if (p.ks == 1 || cap_blocks * SSPB >= p.ks) break;
        }
        const int unit = std::max(p.ks, SSPB);  // (both are powers of two)
        p.blocks = cap_blocks * SSPB / unit * unit / SSPB;
        p.lds = GEMV_SUM_BYTES + p.x_off + (size_t)p.blocks * bp * 1024;
    }
    const int rw = p.nw / p.ks;
    p.ngroups = (int)cdiv(N, 16 * p.rg * rw);
    // resident workgroups: 16 waves and 160 KB of LDS per compute unit, 256 compute units
    const int per_cu = std::max(1, std::min(16 / p.nw, (int)(kLds / p.lds)));
    // A roomy form runs one workgroup to a compute unit.  Where there are more of them than compute units and two would fit, it
    // is held to 128 registers at int3 with one row group (K is cut into eight, a second round is a cold start: 6000 x 4096,
    // B = 4 13.3 -> 10.7 us, 4112 x 4096 12.2 -> 9.8), and at int2 and int6 where rows are short and the main loop little of the
    // work (65600 x 1152 int2, B = 5 16.0 -> 14.5 us, 72704 x 512 int6, B = 1 18.0 -> 16.7; but 70656 x 2048 int6 44.5 -> 45.8, 70000 x 2944 int2, B = 8 26.5 -> 27.7); at int3
    // with two row groups the spills cost more than the second round (65600 x 1024 17.3 and 18.3 us, 73728 x 4608 49.9 and 59.1).
    // Workgroups of sixteen waves are bounded by 1024 threads in any case.
    const bool pairs = per_cu > 1 && p.ngroups > 256;
    p.tight = p.nw > 8 || (pairs && (p.rg == 1 || (r == 6 && lines <= 8) || (r == 2 && lines <= 5)));
    const int capacity = 256 * per_cu;  // (a workgroup too many for a roomy form starts when a compute unit is free)
    const int rounds = (p.ngroups + capacity - 1) / capacity;
    p.grid = (p.ngroups + rounds - 1) / rounds;
    return p;
}

// ============================================================================================
// decode GEMV with K split over workgroups (mq_gemv_reg.hip)
// ============================================================================================
// Workgroups of four waves (a slice of nl lines of a row each, `groups` of them side by side), every wave visiting ch blocks of 16
// rows; about one workgroup per compute unit (measured best on 4096 x 14336 and 4608 x 36864 at B = 8 and 16: 13 us against 25, 25
// against 94; two to four per compute unit cost 10-35 % more, their activation loads grow with the number of workgroups).
// Used for long rows and few of them: at least four groups of slices and at most 8192 rows; elsewhere the one-kernel
// forms are level or faster (4096 x 4096, 14336 x 4096 and taller: 1.0-1.5x the time).
struct GemvSplitPlan {
    int groups, nl, nsl, ks;   // groups == 0: the form is not used
    int depth, ch, grid;       // depth: tiles in a wave's ring; 0: the form does not fit
    size_t lds;
};
// How K is cut (all that the size of the workspace depends on).
inline GemvSplitPlan gemv_split_cut(int64_t B, int64_t N, int64_t KB, int r) {
    GemvSplitPlan p{};
    if (B <= 4 || (r != 2 && r != 4) || (KB & 127) != 0 || N > 8192) return p;
    const int64_t lines = KB >> 7;
    p.nl = r == 4 && lines % 2 == 0 ? 2 : 1;
    const int64_t nsl = lines / p.nl, groups = cdiv(nsl, 4);
    if (groups < 4) return p;
    p.nsl = (int)nsl;
    p.ks = 4;
    p.groups = (int)groups;
    return p;
}
// The ring is the deepest that fits next to the partial results, one workgroup to a compute unit: with four waves there three
// int4 tiles each are not enough in flight (4096 x 14336, B = 16: 16.0 us with three, 14.9 with six, 14.8 with eight; 4608 x
// 36864: 31.2, 28.7, 28.8).  An int2 tile takes twice as long to work on (13.7, 14.0, 14.1; 2304 x 9216 at B = 8 9.3, 9.4, 9.4).
// A shorter ring is still far better than the kernel that does not split K: 8192 x 28672, B = 16 32.2 us with four tiles, 35.2 with
// three, 50.2 there; 7168 x 36864 38.2 with three, 100.0; 4608 x 26880 29.8, 77.9 (8192 x 14080: 25.7 and 30.6, but 23.6 and 21.9 at B = 5).
inline GemvSplitPlan make_gemv_split_plan(int64_t B, int64_t N, int64_t KB, int r) {
    GemvSplitPlan p = gemv_split_cut(B, N, KB, r);
    if (p.groups == 0 || N * KB > 0x7FFFFFFFll) return p;
    const int nrb = (int)cdiv(N, 16), row_groups = std::max(1, 256 / p.groups);
    p.ch = (nrb + row_groups - 1) / row_groups;
    p.grid = (nrb + p.ch - 1) / p.ch;
    for (int depth : {6, 4, 3}) {
        if (r == 2 && depth > 3) continue;
        p.lds = (size_t)p.ks * 128 + (size_t)p.ks * depth * GEMV_TILE + (size_t)p.ks * p.ch * 1024;
        if (p.lds <= 160 * 1024) {
            p.depth = depth;
            break;
        }
    }
    return p;
}

}  // namespace mq
