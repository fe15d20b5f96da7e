// Internal interface of the linear-layer kernels (not part of the public ABI): tile loads, code conversions, and the
// main loop that the forward kernels share.
#pragma once

#include <type_traits>

#include "mq_gemv.h"

namespace mq {

typedef __attribute__((address_space(3))) void *lds_ptr;

constexpr uint32_t kOOB = 0x80000000u;   // buffer offset beyond any descriptor built here
constexpr uint32_t kMagic128 = 0x43004300u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, uint64_t bytes) {
    const uint32_t rec = bytes > 0x7FFFFFFFull ? 0x7FFFFFFFu : (uint32_t)bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)rec, 0x00020000);
}

// All but this wave's newest N global loads have landed and all but its newest L LDS reads are done, then the workgroup
// meets: after it the tiles of the other waves are in LDS too, and the buffer of the previous stage may be filled again (the L
// newest reads of a wave are those of the stage that follows; LDS reads are done in their order).  Not __syncthreads(), whose
// fence waits for every load in flight, direct-to-LDS loads being writes to LDS: wherever the compiler saw loads before a
// barrier (all prologues, two of the three stages of a channel tile in dX) the two stages that should have stayed on their
// way were drained.  14336 x 3584, 8192 tokens, r = 8/4/2: dX 2122 -> 2052 us, forward with the objective 2103 -> 2076 us.
template <int N, int L>
__device__ __forceinline__ void stage_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(%1)\n\ts_barrier" ::"n"(N), "n"(L) : "memory");
}

__device__ __forceinline__ void wait_vm0() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ f32x16 mfma32(const u32x4 &a, const u32x4 &b, const f32x16 &c) {
    Frag8 fa, fb;
    fa.u = a;
    fb.u = b;
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.b, fb.b, c, 0, 0, 0);
}

// ---- LDS tiles ------------------------------------------------------------------------------
// bf16 tile: ROWS x 64 elements, 128-byte rows of eight 16-byte chunks; chunk c of row r is stored
// at chunk position c ^ ((r >> 1) & 7).  u8 tile: ROWS x 64 bytes, four chunks per row; chunk c of
// row r at position c ^ ((r >> 2) & 3).  The LDS has 64 four-byte banks and serves a 16-byte read
// sixteen lanes at a time, so sixteen consecutive rows must land on sixteen distinct 16-byte bank
// groups of a 256-byte window; both swizzles do that (measured: same rate as a contiguous read).  A direct-to-LDS load writes lane l of a wave at base + 16 l, so the swizzle is
// applied by choosing which global chunk each lane fetches.

// Per-lane byte offset (row * ld_bytes + chunk * 16) of instruction `inst` of this wave for a bf16
// tile, and the element column of the chunk (for the tail predicate).
template <int NWAVES>
__device__ __forceinline__ void bf16_tile_lane(int wave, int lane, int inst, uint32_t ld_bytes,
                                               uint32_t &voff, int &col) {
    const int slot = (wave + inst * NWAVES) * 64 + lane;
    const int row = slot >> 3, p = slot & 7, c = p ^ ((row >> 1) & 7);
    voff = (uint32_t)row * ld_bytes + (uint32_t)c * 16u;
    col = c * 8;
}
template <int NWAVES>
__device__ __forceinline__ void u8_tile_lane(int wave, int lane, int inst, uint32_t ld_bytes,
                                             uint32_t &voff, int &col) {
    const int slot = (wave + inst * NWAVES) * 64 + lane;
    const int row = slot >> 2, p = slot & 3, c = p ^ ((row >> 2) & 3);
    voff = (uint32_t)row * ld_bytes + (uint32_t)c * 16u;
    col = c * 16;
}

// ---- code -> bf16 operand conversion -----------------------------------------------------------
// r-bit slice of section 3.2 as bf16(128 + code): the kernels' convert_piece, two codes at a time.
struct SliceParam {  // wave-uniform per bit-width
    uint32_t half2;  // half (<< 8 unless EP) in both 16-bit lanes
    uint32_t sh;     // shift that leaves the code
};

template <bool EP>
__device__ __forceinline__ SliceParam slice_param(int r) {
    const uint32_t s = 8 - r, half = (1u << s) >> 1;
    SliceParam p;
    if constexpr (EP) {
        p.half2 = half | (half << 16);
        p.sh = s;
    } else {
        p.half2 = (half << 8) | (half << 24);
        p.sh = s + 8;
    }
    return p;
}

// ============================================================================================
// forward
// ============================================================================================
struct FwdArgs {
    const uint16_t *X;
    const uint8_t *Q;
    const float *alpha, *zero, *rowsum;
    uint16_t *Y[3];
    int M, N, K;
    int r[3];  // bit-width per slot; slot 0 is the r = 8 slot when HAS8
    int tiles_m, tiles_n;
    // LOSS kernels only (slot order as Y): the L2 objective is evaluated on the rounded outputs
    // while they sit in the staging tiles.  Y[i] may then be NULL (that output is not stored).
    const uint16_t *T;
    uint16_t *dY[3];
    int teacher[3];  // slot of the teacher, or -1 for the target T
    float coef[3];   // lambda_i * 2 / (M N)
    int mix;
    float *partial;  // [workgroup][4] sums of squared differences
    const float *bias;  // [N] added to every output before it is rounded, or null
    // plain kernels only: the layer is the stacked gate / up projection of a gated unit (channels (g, u) pairs)
    // and A[i] [M, N / 2] receives act(g) u of the rounded outputs; gate = 0 none, 1 GELU-tanh, 2 SiLU
    uint16_t *A[3];
    int gate;
};

// The contraction of one workgroup: acc[i][j] = sum over k in [64 kt0, k_end) of code_i[channels of this wave][k] *
// X[tokens m0 + 32 j ..][k], for all bit-widths i and token blocks j of the tile at (m0, n0).  Four waves; wave w owns
// channels [32 w, 32 w + 32) of the tile for all its tokens.  ROWSUM: also rsum[j] += this thread's share (chunk t % 8 of
// row t / 8) of sum_k X for the token blocks in rs_mask.
template <int NR, bool HAS8, bool EP, int MB, bool ROWSUM>
__device__ __forceinline__ void fwd_main_loop(const FwdArgs &a, uint8_t *smem, int m0, int n0, int kt0, int nkt, int k_end,
                                              f32x16 (&acc)[NR][MB], float (&rsum)[MB], uint32_t rs_mask) {
    constexpr int BM = 32 * MB;
    constexpr int X_TILE = BM * 128;
    constexpr int STAGE = X_TILE + FWD_Q_TILE;
    constexpr int LPS = MB + 2;  // direct-to-LDS loads per wave and stage
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, l32 = lane & 31;

    const __amdgpu_buffer_rsrc_t rX = make_rsrc(a.X + (size_t)m0 * a.K, (uint64_t)(a.M - m0) * a.K * 2);
    const __amdgpu_buffer_rsrc_t rQ = make_rsrc(a.Q + (size_t)n0 * a.K, (uint64_t)(a.N - n0) * a.K);

    // global -> LDS: lane offsets of the wave's first X / Q instruction; instruction i is 32 (X) or
    // 64 (Q) rows further down with the same chunk
    uint32_t xoff0, qoff0;
    int xcol, qcol;
    bf16_tile_lane<4>(wave, lane, 0, (uint32_t)a.K * 2u, xoff0, xcol);
    u8_tile_lane<4>(wave, lane, 0, (uint32_t)a.K, qoff0, qcol);
    const uint32_t xstep = 32u * (uint32_t)a.K * 2u, qstep = 64u * (uint32_t)a.K;

    // Stage kt -> LDS buffer kt % 4, as MB + 2 loads per wave (MB of X, then 2 of Q).  Branch-free:
    // a stage past k_end (or a chunk past it in the last stage) is requested at an out-of-range offset, which the buffer unit answers with zeros without touching memory, so
    // the number of loads in flight is the same in every iteration.
    auto issue_one = [&](int kt, int i) {
        const int k0 = (kt0 + kt) * BKT;
        uint8_t *xs = smem + (kt & 3) * STAGE;
        if (i < MB) {
            // (an out-of-range base stays out of range: kOOB + i * xstep < 2^32 for every legal K)
            const uint32_t xb = (k0 + xcol < k_end) ? xoff0 + (uint32_t)k0 * 2u : kOOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rX, (lds_ptr)(xs + (wave + i * 4) * 1024), 16,
                                                     xb + (uint32_t)i * xstep, 0, 0, 0);
        } else {
            const uint32_t qb = (k0 + qcol < k_end) ? qoff0 + (uint32_t)k0 : kOOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rQ, (lds_ptr)(xs + X_TILE + (wave + (i - MB) * 4) * 1024), 16,
                                                     qb + (uint32_t)(i - MB) * qstep, 0, 0, 0);
        }
    };
    auto issue = [&](int kt) {
#pragma unroll
        for (int i = 0; i < MB + 2; ++i) issue_one(kt, i);
    };

    // LDS fragment addresses (byte offsets inside a stage)
    const int nl = wave * 32 + l32;
    const uint32_t qa0 = X_TILE + nl * 64 + ((h ^ ((nl >> 2) & 3)) << 4);
    const uint32_t qa1 = X_TILE + nl * 64 + (((h + 2) ^ ((nl >> 2) & 3)) << 4);
    uint32_t xa[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int cx = 2 * h + 4 * (t >> 1) + (t & 1);
        xa[t] = l32 * 128 + ((cx ^ ((l32 >> 1) & 7)) << 4);
    }

    SliceParam sp[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) sp[i] = slice_param<EP>(a.r[i]);

    // Dword w (two consecutive k) of the code operand of slot i, from the 8 code bytes (d0, d1).
    auto convert_piece = [&](int i, int w, uint32_t d0, uint32_t d1) -> uint32_t {
        const uint32_t d = w < 2 ? d0 : d1;
        if (HAS8 && i == 0) {
            const float lo = (w & 1) ? (float)((d >> 16) & 0xFFu) : (float)(d & 0xFFu);
            const float hi = (w & 1) ? (float)(d >> 24) : (float)((d >> 8) & 0xFFu);
            return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
        }
        if constexpr (EP) {
            const uint32_t placed = __builtin_amdgcn_perm(0u, d, (w & 1) ? 0x0C030C02u : 0x0C010C00u);
            return (((placed + sp[i].half2) >> sp[i].sh) & 0x00FF00FFu) | kMagic128;
        } else {
            const uint32_t placed = __builtin_amdgcn_perm(0u, d, (w & 1) ? 0x030C020Cu : 0x010C000Cu);
            u16x2 t = __builtin_elementwise_add_sat(__builtin_bit_cast(u16x2, placed),
                                                    __builtin_bit_cast(u16x2, sp[i].half2));
            const unsigned short s16 = (unsigned short)sp[i].sh;
            t = t >> u16x2{s16, s16};
            return __builtin_bit_cast(uint32_t, t) | kMagic128;
        }
    };

#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    issue(0);
    issue(1);
    issue(2);
    // stage 0 must have landed before the first operand fetch; stages 1 and 2 may stay in flight
    stage_barrier<2 * LPS, 0>();

    u32x4 xf[MB];      // activation operands of the current k step (refilled as soon as they are consumed)
    u32x4 raw[2];      // 32 code bytes of this lane's channel: four k steps of one stage
    u32x4 wf[NR];      // code operands of the current k step
    raw[0] = *reinterpret_cast<const u32x4 *>(smem + qa0);
    raw[1] = *reinterpret_cast<const u32x4 *>(smem + qa1);
#pragma unroll
    for (int j = 0; j < MB; ++j) xf[j] = *reinterpret_cast<const u32x4 *>(smem + xa[0] + j * 4096);
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int w = 0; w < 4; ++w) wf[i][w] = convert_piece(i, w, raw[0][0], raw[0][1]);

    // One stage of 64 k: four 16-wide steps of NR * MB MFMAs.  A wave issues in order, so whatever
    // is queued behind an MFMA that waits for the matrix pipe waits with it; the other work of a
    // step is therefore cut into one small group per MFMA, fenced so that the compiler keeps it
    // there:  group q < MB requests operand block q of step t + 1 from LDS (it then has the rest
    // of the step to arrive), groups 1 .. 4 NR each produce one dword of the next code operands,
    // the last groups of step 0 issue the global loads of stage kt + 3, and step 2 fetches the
    // code bytes of the next stage.  MORE (compile time): there is a next stage.
    auto tile = [&](auto more_tag, int kt) {
        constexpr bool MORE = decltype(more_tag)::value;
        constexpr int NM = NR * MB;
        constexpr int CQ = 4 * NR + 1 <= NM ? 1 : 0;                // first group that carries a conversion
        constexpr int PPG = (4 * NR + NM - CQ - 1) / (NM - CQ);     // conversions per group (1 from MB = 4 on)
        constexpr int LPG = (LPS + NM - 1) / NM;  // global loads per group in step 0
        const uint8_t *cur = smem + (kt & 3) * STAGE;
        const uint8_t *nxt = smem + ((kt + 1) & 3) * STAGE;
        u32x4 rawn[2];
        if constexpr (ROWSUM) {
            // thread t adds chunk t % 8 of row t / 8 of the token blocks this workgroup sums (zeros past M and k_end)
#pragma unroll
            for (int j = 0; j < MB; ++j)
                if (rs_mask & (1 << j)) {
                    const u32x4 v = *reinterpret_cast<const u32x4 *>(cur + j * 4096 + threadIdx.x * 16);
#pragma unroll
                    for (int w = 0; w < 4; ++w) rsum[j] += bf16_lo(v[w]) + bf16_hi(v[w]);
                }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bool pre = t < 3 || MORE;  // is there a next step
            const uint8_t *src = t < 3 ? cur + xa[(t + 1) & 3] : nxt + xa[0];
            // code bytes of the next step
            uint32_t d0 = t == 3 ? rawn[0][0] : (t + 1 < 2 ? raw[0][2 * (t + 1)] : raw[1][2 * (t + 1 - 2)]);
            uint32_t d1 = t == 3 ? rawn[0][1] : (t + 1 < 2 ? raw[0][2 * (t + 1) + 1] : raw[1][2 * (t + 1 - 2) + 1]);
            // pin the conversions of this step to this step (the optimizer would otherwise collect
            // them across the loop back-edge)
            if (pre) asm volatile("" : "+v"(d0), "+v"(d1));
            u32x4 xfn[MB];
            u32x4 wfn[NR];
#pragma unroll
            for (int q = 0; q < NM; ++q) {
                const int j = q / NR, i = q % NR;
                acc[i][j] = mfma32(wf[i], xf[j], acc[i][j]);
                if (pre && q < MB) xfn[q] = *reinterpret_cast<const u32x4 *>(src + q * 4096);
                if (pre && q >= CQ) {
#pragma unroll
                    for (int u = 0; u < PPG; ++u) {
                        const int pc = (q - CQ) * PPG + u;
                        if (pc < 4 * NR) {
                            uint32_t piece = convert_piece(pc / 4, pc % 4, d0, d1);
                            asm volatile("" : "+v"(piece));  // keeps the conversion inside this group
                            wfn[pc / 4][pc % 4] = piece;
                        }
                    }
                }
                if (MORE && t == 2) {
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        if (q == (NM > 2 ? NM - 2 + u : NM - 1)) rawn[u] = *reinterpret_cast<const u32x4 *>(nxt + (u ? qa1 : qa0));
                }
                if (MORE && t == 0) {
#pragma unroll
                    for (int u = 0; u < LPG; ++u) {
                        const int ld = (NM - 1 - q) * LPG + u;  // the last groups carry the loads
                        if (ld < LPS) issue_one(kt + 3, ld);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (pre) {
#pragma unroll
                for (int i = 0; i < NR; ++i) wf[i] = wfn[i];
#pragma unroll
                for (int j = 0; j < MB; ++j) xf[j] = xfn[j];
            }
        }
        if (MORE) {
            raw[0] = rawn[0];
            raw[1] = rawn[1];
        }
    };

    for (int kt = 0; kt + 1 < nkt; ++kt) {
        // Stage kt + 1 must be resident for the operand prefetch at the end of this iteration; the
        // loads of stage kt + 2 may stay in flight.  After the barrier every wave is done with
        // stage kt - 1, whose buffer stage kt + 3 reuses.
        stage_barrier<LPS, MB>();
        tile(std::true_type{}, kt);
    }
    tile(std::false_type{}, nkt - 1);
    wait_vm0();  // zero-fill loads of dead stages must not land in the staging area below
}

// the forward for few tokens (mq_linear_split.hip): its cut, remembered, and its launches (plan.mb != 0)
FwdSplitPlan fwd_split_plan(int64_t M, int64_t N, int64_t K, int nr);
mq_status launch_fwd_split(const FwdArgs &f, const FwdSplitPlan &plan, int nr, bool has8, bool ep, bool loss, float *part,
                           float *rs_part, hipStream_t st, int64_t *blocks);

// ============================================================================================
// backward dX, forward at one bit-width (mq_linear_wide.hip)
// ============================================================================================
struct DxArgs {
    const uint16_t *As[3];  // [M, N] bf16, slot order (the r = 8 slot first when HAS8)
    const uint8_t *QT;      // [K, N] u8
    const float *cvec;      // [nsplit][M]: partial sums of c[m] over column ranges
    int nsplit;
    uint16_t *dX;           // [M, K] bf16
    int M, N, K;
    int r[3];               // bit-width per slot
    int tiles_m, tiles_k;
    int splits;             // ranges of n per tile
    float *part;            // splits > 1: fp32 accumulators, [split][tile][k block][token block][g][256] quads
};

DxPlan dx_plan(int64_t M, int64_t N, int64_t K, int nr);
// the forward at one bit-width (plain or gated), mb as fwd_wide_mb has chosen it
mq_status launch_fwd_wide(const FwdArgs &f, int mb, bool has8, bool ep, hipStream_t st);
mq_status launch_dx(DxArgs d, const DxPlan &plan, int nr, bool has8, bool ep, hipStream_t st);

}  // namespace mq
