// The products whose tiles are 256 code rows wide: dX of the straight-through backward, with its contraction cut into ranges
// for the sizes whose tiles leave compute units idle, and the forward at one bit-width.
#include <algorithm>

#include "mq_linear.h"

namespace mq {

// ============================================================================================
// backward dX: dX[m, k] = sum_i sum_n As_i[m, n] * V_i[n, k] - c[m], V_i = the bf16 operand of slot i
// Rows of the matrix-core product are k (from the transposed codes QT[K, N]), columns are tokens,
// the contraction runs over n and, within each n tile, over the bit-widths.
// ============================================================================================
static_assert(dx_lds(DX_MB) >= 32 * DX_MB * DX_OS && dx_lds(1) >= 32 * DX_OS, "the staging tile has to fit");

// Same pipeline as the forward kernel (one wave per SIMD, four LDS stages, one small fenced group
// of operand work per MFMA), with the roles changed: a stage is one 64-wide tile of n for ONE
// bit-width, i.e. the gradient operand As_slot[tokens, n tile] and the transposed codes
// QT[k rows, n tile]; the NRS bit-widths of an n tile follow each other and all accumulate into the
// same accumulators.  Wave w owns k rows [64 w, 64 w + 64) for all 32 MB tokens of the tile.  The
// stage loop is unrolled over the bit-widths so that the kind of code conversion is a compile-time
// property of each copy of the stage body.
//
template <int NRS, bool HAS8, bool LAST2, bool EP, int MB>
__device__ __forceinline__ void wide_main_loop(const DxArgs &a, uint8_t *smem, int m0, int k0, int nt0, int nt1, f32x4 (&acc)[2 * DX_RB][2 * MB]) {
    constexpr int RB = 2 * DX_RB;        // 16-row blocks per wave
    constexpr int A_TILE = MB * 4096;
    constexpr int STAGE = A_TILE + DX_Q_TILE;
    constexpr int QL = DX_BK / 64;       // direct-to-LDS loads per wave and stage for the codes (16 rows each)
    constexpr int LPS = MB + QL;         // loads per wave and stage
    constexpr int NM = 2 * MB * RB;      // MFMAs per 32-wide step
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g4 = lane >> 4, l16 = lane & 15;

    const int n_end = min(a.N, nt1 * BKT);

    __amdgpu_buffer_rsrc_t rA[NRS];
#pragma unroll
    for (int i = 0; i < NRS; ++i) rA[i] = make_rsrc(a.As[i] + (size_t)m0 * a.N, (uint64_t)(a.M - m0) * a.N * 2);
    const __amdgpu_buffer_rsrc_t rQ = make_rsrc(a.QT + (size_t)k0 * a.N, (uint64_t)(a.K - k0) * a.N);

    uint32_t aoff0, qoff0;
    int acol, qcol;
    bf16_tile_lane<4>(wave, lane, 0, (uint32_t)a.N * 2u, aoff0, acol);
    u8_tile_lane<4>(wave, lane, 0, (uint32_t)a.N, qoff0, qcol);
    const uint32_t astep = 32u * (uint32_t)a.N * 2u, qstep = 64u * (uint32_t)a.N;

    // load i of stage (n tile nt, bit-width slot) into LDS buffer `buf`; out-of-range requests
    // (a tile past the range) are answered with zeros, so the loads in flight are the same every stage
    auto issue_one = [&](int nt, auto slot_tag, int buf, int i) {
        constexpr int SLOT = decltype(slot_tag)::value;
        const int n0 = nt * BKT;
        uint8_t *as = smem + buf * STAGE;
        if (i < MB) {
            const uint32_t ab = (n0 + acol < n_end) ? aoff0 + (uint32_t)n0 * 2u : kOOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rA[SLOT], (lds_ptr)(as + (wave + i * 4) * 1024), 16,
                                                     ab + (uint32_t)i * astep, 0, 0, 0);
        } else {
            // The code bytes of an n tile are fetched with its first bit-width only: the other bit-widths
            // of the tile slice the same bytes, which the lanes then still hold in registers.  Their
            // requests go out of range (no traffic) so that every stage has the same number of loads.
            const uint32_t qb = (SLOT == 0 && n0 + qcol < n_end) ? qoff0 + (uint32_t)n0 : kOOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rQ, (lds_ptr)(as + A_TILE + (wave + (i - MB) * 4) * 1024), 16,
                                                     qb + (uint32_t)(i - MB) * qstep, 0, 0, 0);
        }
    };

    // LDS fragment addresses (byte offsets inside a stage); the order of the contraction is that of fwd_main_loop
    const int kl = wave * (16 * RB) + l16;
    const int gc = group_chunk(g4);
    const uint32_t qa = A_TILE + kl * 64 + ((gc ^ ((kl >> 2) & 3)) << 4);   // + 1024 per block of 16 rows
    uint32_t xa[2];                                                         // + 2048 per block of 16 tokens
#pragma unroll
    for (int t = 0; t < 2; ++t) xa[t] = l16 * 128 + (((2 * gc + t) ^ ((l16 >> 1) & 7)) << 4);

    SliceParam sp[NRS];
#pragma unroll
    for (int i = 0; i < NRS; ++i) sp[i] = slice_param<EP>(a.r[i]);

#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int tb = 0; tb < 2 * MB; ++tb) acc[rb][tb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // prologue: stages 0, 1, 2 (n tile nt0 + st / NRS, bit-width st % NRS)
    {
        auto issue_stage = [&](auto st_tag) {
            constexpr int ST = decltype(st_tag)::value;
#pragma unroll
            for (int i = 0; i < LPS; ++i) issue_one(nt0 + ST / NRS, std::integral_constant<int, ST % NRS>{}, ST & 3, i);
        };
        issue_stage(std::integral_constant<int, 0>{});
        issue_stage(std::integral_constant<int, 1>{});
        issue_stage(std::integral_constant<int, 2>{});
    }
    stage_barrier<2 * LPS, 0>();

    constexpr int XS = MB <= 2 ? 2 : 1;   // sets of gradient operands (see fwd_main_loop)
    u32x4 xf[XS][2 * MB];
    u32x4 raw[RB];        // the sixteen code bytes of this lane's rows: both steps of one stage
    u32x4 wf[2][RB];      // code operands of the two steps of a stage
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) raw[rb] = *reinterpret_cast<const u32x4 *>(smem + qa + rb * 1024);
#pragma unroll
    for (int tb = 0; tb < 2 * MB; ++tb) xf[0][tb] = *reinterpret_cast<const u32x4 *>(smem + xa[0] + tb * 2048);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) wf[0][rb] = convert_eight<code_kind(HAS8, LAST2 && NRS == 1), EP>(raw[rb][0], raw[rb][1], sp[0]);

    // One stage: two 32-wide steps, the other work in between the MFMAs as in fwd_main_loop.  st = index of this stage; the loads
    // issued in step 0 fetch stage st + 3.
    auto tile = [&](auto slot_tag, int st, int nt) {
        constexpr int SLOT = decltype(slot_tag)::value;
        constexpr int NEXT = (SLOT + 1) % NRS;
        const uint8_t *cur = smem + (st & 3) * STAGE;
        const uint8_t *nxt = smem + ((st + 1) & 3) * STAGE;
        u32x4 rawn[RB];
        static_for<2>([&](auto t_tag) {
            constexpr int t = decltype(t_tag)::value;
            constexpr int CSLOT = t == 0 ? SLOT : NEXT;       // bit-width of the operands that are converted
            constexpr bool IS8 = HAS8 && CSLOT == 0, IS2 = LAST2 && CSLOT == NRS - 1;
            // (the code bytes of a new n tile are read; those of its other bit-widths are at hand)
            constexpr StepSchedule<NM, RB, 2 * MB, 2 * RB, 1, IS8, t, LPS, NRS == 3 && MB >= 4, NEXT == 0 ? RB : 0, XS == 1,
                                   false, 2> plan;
            const uint8_t *src = t == 0 ? cur + xa[1] : nxt + xa[0];
            uint32_t tmp[plan.width][4];
            static_for<NM>([&](auto q_tag) {
                constexpr int q = decltype(q_tag)::value, tb = q / RB, rb = q % RB;
                mfma16_acc(acc[rb][tb], wf[t][rb], xf[t % XS][tb]);
                if constexpr (XS == 2 && q < 2 * MB) xf[1 - t % XS][q] = *reinterpret_cast<const u32x4 *>(src + q * 2048);
                if constexpr (XS == 1 && rb == RB - 1) xf[0][tb] = *reinterpret_cast<const u32x4 *>(src + tb * 2048);
                static_for<plan.code[q + 1] - plan.code[q]>([&](auto u_tag) {
                    constexpr int e = plan.code[q] + decltype(u_tag)::value;
                    rawn[e] = *reinterpret_cast<const u32x4 *>(nxt + qa + e * 1024);
                });
                static_for<plan.conv[q + 1] - plan.conv[q]>([&](auto u_tag) {
                    constexpr int c = plan.conv[q] + decltype(u_tag)::value, crb = plan.pair[c] / 2, half = plan.pair[c] % 2;
                    u32x4 &out = wf[1 - t][crb];
                    uint32_t lo = out[2 * half], hi = out[2 * half + 1];
                    convert_step<code_kind(IS8, IS2), EP, plan.step[c]>(t == 0 ? raw[crb][2 + half] : NEXT == 0 ? rawn[crb][half] : raw[crb][half], sp[CSLOT],
                                                        tmp[plan.at[c]], lo, hi);
                    if constexpr (plan.step[c] == (IS8 ? 2 : 3)) {
                        out[2 * half] = lo;
                        out[2 * half + 1] = hi;
                    }
                });
                static_for<plan.load[q + 1] - plan.load[q]>([&](auto u_tag) {
                    issue_one(nt + (SLOT + 3) / NRS, std::integral_constant<int, (SLOT + 3) % NRS>{}, (st + 3) & 3,
                              plan.first_load + plan.load[q] + decltype(u_tag)::value);
                });
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        mfma16_settle();
        if constexpr (NEXT == 0) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) raw[rb] = rawn[rb];
        }
    };
    auto stage = [&](auto slot_tag, int st, int nt) {
        // stage st + 1 must be resident (operand prefetch inside this stage); the loads of
        // stage st + 2 may stay in flight; after the barrier the buffer of stage st - 1 is free
        stage_barrier<LPS, 2 * MB>();
        tile(slot_tag, st, nt);
    };

    int st = 0;
    for (int nt = nt0; nt < nt1; ++nt) {
        stage(std::integral_constant<int, 0>{}, st++, nt);
        if constexpr (NRS > 1) stage(std::integral_constant<int, 1>{}, st++, nt);
        if constexpr (NRS > 2) stage(std::integral_constant<int, 2>{}, st++, nt);
    }
    wait_vm0();  // zero-fill loads of dead stages must not land in the staging area below
}

// a.splits > 1: workgroup (range, tile) contracts one range of n tiles and leaves its fp32 accumulators in a.part in the
// order its lanes hold them (each store a whole 1 KB per wave); dx_finish_kernel adds the ranges.
template <int NRS, bool HAS8, bool LAST2, bool EP, int MB>
__global__ __launch_bounds__(256) void dx_kernel(DxArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    constexpr int RB = 2 * DX_RB, BM = 32 * MB;  // 16-row blocks per wave
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g4 = lane >> 4, l16 = lane & 15;

    const int tiles = a.tiles_m * a.tiles_k;
    const uint32_t wid = xcd_contiguous_id(blockIdx.x, gridDim.x);
    const int split = (int)wid / tiles;
    const uint32_t lid = wid % (uint32_t)tiles;
    const int nnt_all = (a.N + BKT - 1) / BKT;
    const int nt0 = (int)((int64_t)nnt_all * split / a.splits), nt1 = (int)((int64_t)nnt_all * (split + 1) / a.splits);
    constexpr int GROUP = 4;
    const int width = GROUP * a.tiles_k;
    const int first_m = (int)(lid / width) * GROUP;
    const int gsz = min(a.tiles_m - first_m, GROUP);
    const int tm = first_m + (int)(lid % width) % gsz;
    const int tk = (int)(lid % width) / gsz;
    const int m0 = tm * BM, k0 = tk * DX_BK;

    f32x4 acc[RB][2 * MB];
    wide_main_loop<NRS, HAS8, LAST2, EP, MB>(a, smem, m0, k0, nt0, nt1, acc);

    if (a.splits > 1) {
        f32x4 *dst = reinterpret_cast<f32x4 *>(a.part) + ((size_t)split * tiles + lid) * (RB * 2 * MB * 256) + threadIdx.x;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int tb = 0; tb < 2 * MB; ++tb)
                if (m0 + 16 * tb < a.M) dst[(rb * 2 * MB + tb) * 256] = acc[rb][tb];  // (dx_finish_kernel reads no other)
        return;
    }

    // ---- epilogue: rows of the product are k, columns tokens; dX = acc - c[m] --------------------
    // assembled in LDS as [token][k] bf16 (rows of DX_OS bytes) and stored as whole 512-byte rows
    __syncthreads();
    // c[m] = sum over the column ranges of the prep kernel, in their order.  The partial sums of all the
    // lane's tokens are requested four ranges at a time (one memory round trip per
    // group instead of one per value, which with nothing else to run cost more than the stores).
    float cs[2 * MB];
#pragma unroll
    for (int tb = 0; tb < 2 * MB; ++tb) cs[tb] = 0.f;
    for (int sp0 = 0; sp0 < a.nsplit; sp0 += 4) {
        float part[4][2 * MB];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int tb = 0; tb < 2 * MB; ++tb) {
                const int m = m0 + tb * 16 + l16;
                part[u][tb] = (sp0 + u < a.nsplit && m < a.M) ? a.cvec[(size_t)(sp0 + u) * a.M + m] : 0.f;
            }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int tb = 0; tb < 2 * MB; ++tb) cs[tb] += part[u][tb];
    }
#pragma unroll
    for (int tb = 0; tb < 2 * MB; ++tb) {
        const float c = cs[tb];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int kloc = wave * (16 * RB) + rb * 16 + 4 * g4;
            const f32x4 v = acc[rb][tb];
            *reinterpret_cast<u32x2 *>(smem + (tb * 16 + l16) * DX_OS + kloc * 2) =
                u32x2{pack_bf16x2(v[0] - c, v[1] - c), pack_bf16x2(v[2] - c, v[3] - c)};
        }
    }
    __syncthreads();
    constexpr int CPR = DX_BK / 8;  // 16-byte chunks per row
#pragma unroll
    for (int it = 0; it < BM * CPR / 256; ++it) {
        const int c = it * 256 + threadIdx.x;
        const int row = c / CPR, ch = c % CPR;
        const int m = m0 + row, k = k0 + ch * 8;
        if (m < a.M && k < a.K) {
            const uint8_t *src = smem + row * DX_OS + ch * 16;
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(src), reinterpret_cast<u32x4 *>(a.dX + (size_t)m * a.K + k));
        }
    }
#else
    (void)a;
#endif
}

// Adds the ranges of the contraction in their order and finishes dX.  Workgroup = (tile, 32 tokens, 32 rows of k of
// one wave of dx_kernel): its four waves take the four 16 x 16 blocks and write 64 contiguous bytes of 32 tokens.
__global__ __launch_bounds__(256) void dx_finish_kernel(DxArgs a, int mb) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g4 = lane >> 4, l16 = lane & 15;
    const int w = blockIdx.x & 3, rest = (int)(blockIdx.x >> 2) / DX_RB;
    const int rb = (int)(blockIdx.x >> 2) % DX_RB * 2 + (wave & 1), tb = rest % mb * 2 + (wave >> 1), tile = rest / mb;
    const int tiles = a.tiles_m * a.tiles_k;
    constexpr int GROUP = 4;   // tile order of dx_kernel
    const int width = GROUP * a.tiles_k;
    const int first_m = tile / width * GROUP;
    const int gsz = min(a.tiles_m - first_m, GROUP);
    const int tm = first_m + tile % width % gsz, tk = tile % width / gsz;
    const int m = tm * 32 * mb + tb * 16 + l16, k = tk * DX_BK + w * 32 * DX_RB + rb * 16 + 4 * g4;
    if (m >= a.M || k >= a.K) return;

    const size_t step = (size_t)tiles * DX_RB * mb * 1024;
    const f32x4 *src = reinterpret_cast<const f32x4 *>(a.part) + (((size_t)tile * 2 * DX_RB + rb) * 2 * mb + tb) * 256 + w * 64 + lane;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < a.splits; p0 += 4) {  // the loads of four ranges are in flight together
        f32x4 v[4];
#pragma unroll
        for (int p = 0; p < 4; ++p)
            v[p] = p0 + p < a.splits ? __builtin_nontemporal_load(src + (p0 + p) * step) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < 4; ++p) sum += v[p];
    }
    float c = 0.f;
    for (int s0 = 0; s0 < a.nsplit; s0 += 4) {
        float v[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) v[p] = s0 + p < a.nsplit ? a.cvec[(size_t)(s0 + p) * a.M + m] : 0.f;
#pragma unroll
        for (int p = 0; p < 4; ++p) c += v[p];
    }
    *reinterpret_cast<u32x2 *>(a.dX + (size_t)m * a.K + k) = u32x2{pack_bf16x2(sum[0] - c, sum[1] - c), pack_bf16x2(sum[2] - c, sum[3] - c)};
}

// ============================================================================================
// forward at one bit-width
// ============================================================================================
// The main loop of dX with other names: Y[m, n] = sum over k of X[m, k] * code[n, k], one bit-width.  With a single bit-width a
// wave of the forward kernel (32 channels) reads one activation operand from LDS per product, 128 bytes per clock and compute
// unit at the matrix-core rate, which is all the LDS delivers; 64 channels per wave halve that.  The order of every sum and the
// arithmetic of the epilogue are those of fwd_kernel.
struct FwdWideArgs {
    DxArgs d;  // As[0] = X [M, K], QT = Q [N, K]; d.N is the contraction length K, d.K the channels N
    const float *alpha, *zero, *rowsum;
    uint16_t *Y, *A;  // A: see FwdArgs; either may be null
    int gate;
};

template <bool HAS8, bool LAST2, bool EP, int MB>
__global__ __launch_bounds__(256) void fwd_wide_kernel(FwdWideArgs w) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const DxArgs &a = w.d;
    constexpr int RB = 2 * DX_RB, BM = 32 * MB;  // 16-row blocks per wave
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g4 = lane >> 4, l16 = lane & 15;

    const uint32_t lid = xcd_contiguous_id(blockIdx.x, gridDim.x);
    constexpr int GROUP = 4;
    const int width = GROUP * a.tiles_k;
    const int first_m = (int)(lid / width) * GROUP;
    const int gsz = min(a.tiles_m - first_m, GROUP);
    const int tm = first_m + (int)(lid % width) % gsz;
    const int tn = (int)(lid % width) / gsz;
    const int m0 = tm * BM, n0 = tn * DX_BK, N = a.K;

    f32x4 acc[RB][2 * MB];
    wide_main_loop<1, HAS8, LAST2, EP, MB>(a, smem, m0, n0, 0, (a.N + BKT - 1) / BKT, acc);

    __syncthreads();  // every wave is done with the operand stages
    float rs[2 * MB];
#pragma unroll
    for (int tb = 0; tb < 2 * MB; ++tb) {
        const int m = m0 + tb * 16 + l16;
        rs[tb] = m < a.M ? w.rowsum[m] : 0.f;
    }
    f32x4 al[RB], ze[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int n = n0 + wave * (16 * RB) + rb * 16 + 4 * g4;
        al[rb] = ze[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (n < N) {
            al[rb] = *reinterpret_cast<const f32x4 *>(w.alpha + n);
            ze[rb] = *reinterpret_cast<const f32x4 *>(w.zero + n);
        }
    }
    const float mult = HAS8 ? 1.0f : (float)(1 << (8 - a.r[0])), offset = HAS8 ? 0.0f : 128.0f * mult;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int nloc = wave * (16 * RB) + rb * 16 + 4 * g4;
#pragma unroll
        for (int tb = 0; tb < 2 * MB; ++tb) {
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float t = (offset + ze[rb][e]) * rs[tb], v = acc[rb][tb][e];
                y[e] = al[rb][e] * (HAS8 ? v - t : __builtin_fmaf(mult, v, -t));
            }
            const u32x2 o = {pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
            *reinterpret_cast<u32x2 *>(smem + (tb * 16 + l16) * DX_OS + nloc * 2) = o;
        }
    }
    __syncthreads();
    constexpr int CPR = DX_BK / 8;  // 16-byte chunks per row
#pragma unroll
    for (int it = 0; it < BM * CPR / 256; ++it) {
        const int c = it * 256 + threadIdx.x;
        const int row = c / CPR, ch = c % CPR;
        const int m = m0 + row, n = n0 + ch * 8;
        if (m < a.M && n < N) {
            const uint8_t *src = smem + row * DX_OS + ch * 16;
            const u32x4 y = *reinterpret_cast<const u32x4 *>(src);
            if (w.Y)
                __builtin_nontemporal_store(y, reinterpret_cast<u32x4 *>(w.Y + (size_t)m * N + n));
            if (w.gate) {
                auto gated = [&](uint32_t pair) {
                    const float g = bf16_lo(pair), u = bf16_hi(pair);
                    return (w.gate == 2 ? silu(g) : gelu_tanh(g)) * u;
                };
                const u32x2 o = {pack_bf16x2(gated(y[0]), gated(y[1])), pack_bf16x2(gated(y[2]), gated(y[3]))};
                __builtin_nontemporal_store(o, reinterpret_cast<u32x2 *>(w.A + (size_t)m * (N >> 1) + (n >> 1)));
            }
        }
    }
#else
    (void)w;
#endif
}

// ---- host side ------------------------------------------------------------------------------------
namespace {

template <bool HAS8, bool LAST2, bool EP, int MB>
mq_status launch_fwd_wide_mb(const FwdWideArgs &w, hipStream_t st) {
    if (!allow_lds<fwd_wide_kernel<HAS8, LAST2, EP, MB>>(dx_lds(MB))) return MQ_ERR_DEVICE;
    fwd_wide_kernel<HAS8, LAST2, EP, MB><<<dim3(w.d.tiles_m * w.d.tiles_k), dim3(256), dx_lds(MB), st>>>(w);
    return launch_status();
}

template <bool HAS8, bool LAST2, bool EP>
mq_status launch_fwd_wide_one(const FwdWideArgs &w, int mb, hipStream_t st) {
    switch (mb) {
        case 3: return launch_fwd_wide_mb<HAS8, LAST2, EP, 3>(w, st);
        case 4: return launch_fwd_wide_mb<HAS8, LAST2, EP, 4>(w, st);
        case 5: return launch_fwd_wide_mb<HAS8, LAST2, EP, 5>(w, st);
        default: return launch_fwd_wide_mb<HAS8, LAST2, EP, 6>(w, st);
    }
}

template <int NRS, bool HAS8, bool LAST2, bool EP, int MB>
mq_status launch_dx_mb(const DxArgs &d, hipStream_t st) {
    // (three bit-widths in tiles of 128 and 160 tokens: 0.9997 times as long with the look-up, 0.977 to 1.016 at 95 sizes)
    constexpr bool LOOKED_UP = LAST2 && !(NRS == 3 && MB >= 4);
    if (!allow_lds<dx_kernel<NRS, HAS8, LOOKED_UP, EP, MB>>(dx_lds(MB))) return MQ_ERR_DEVICE;
    dx_kernel<NRS, HAS8, LOOKED_UP, EP, MB><<<dim3(d.tiles_m * d.tiles_k * d.splits), dim3(256), dx_lds(MB), st>>>(d);
    return launch_status();
}

template <int NRS, bool HAS8, bool LAST2, bool EP>
mq_status launch_dx_form(const DxArgs &d, int mb, hipStream_t st) {
    switch (mb) {
        case 1: return launch_dx_mb<NRS, HAS8, LAST2, EP, 1>(d, st);
        case 2: return launch_dx_mb<NRS, HAS8, LAST2, EP, 2>(d, st);
        case 3: return launch_dx_mb<NRS, HAS8, LAST2, EP, 3>(d, st);
        case 4: return launch_dx_mb<NRS, HAS8, LAST2, EP, 4>(d, st);
        default: return launch_dx_mb<NRS, HAS8, LAST2, EP, 5>(d, st);
    }
}

template <int NRS, bool HAS8, bool EP>
mq_status launch_dx_one(const DxArgs &d, int mb, hipStream_t st) {
    if constexpr (has_last2(NRS, HAS8))
        if (d.r[NRS - 1] == 2) return launch_dx_form<NRS, HAS8, true, EP>(d, mb, st);
    return launch_dx_form<NRS, HAS8, false, EP>(d, mb, st);
}

template <int NRS>
mq_status launch_dx_nrs(const DxArgs &d, int mb, bool has8, bool ep, hipStream_t st) {
    if constexpr (NRS == 1) ep = ep && !has8;  // the code of r = 8 is never rounded up past the byte
    if (has8) {
        if constexpr (NRS > 1)
            if (ep) return launch_dx_one<NRS, true, true>(d, mb, st);
        return launch_dx_one<NRS, true, false>(d, mb, st);
    }
    return ep ? launch_dx_one<NRS, false, true>(d, mb, st) : launch_dx_one<NRS, false, false>(d, mb, st);
}

}  // namespace

DxPlan dx_plan(int64_t M, int64_t N, int64_t K, int nr) { return remembered<DxPlan>(make_dx_plan, M, N, K, nr); }

mq_status launch_fwd_wide(const FwdArgs &f, int mb, bool has8, bool ep, hipStream_t st) {
    FwdWideArgs w{};
    w.d.As[0] = f.X;
    w.d.QT = f.Q;
    w.d.M = f.M;
    w.d.N = f.K;
    w.d.K = f.N;
    w.d.r[0] = f.r[0];
    w.d.tiles_m = (int)cdiv(f.M, 32 * mb);
    w.d.tiles_k = (int)cdiv(f.N, DX_BK);
    w.d.splits = 1;
    w.alpha = f.alpha;
    w.zero = f.zero;
    w.rowsum = f.rowsum;
    w.Y = f.Y[0];
    w.A = f.A[0];
    w.gate = f.gate;
    if (has8) return launch_fwd_wide_one<true, false, false>(w, mb, st);  // the code of r = 8 is never rounded up past the byte
    if (w.d.r[0] == 2) return ep ? launch_fwd_wide_one<false, true, true>(w, mb, st) : launch_fwd_wide_one<false, true, false>(w, mb, st);
    return ep ? launch_fwd_wide_one<false, false, true>(w, mb, st) : launch_fwd_wide_one<false, false, false>(w, mb, st);
}

mq_status launch_dx(DxArgs d, const DxPlan &plan, int nr, bool has8, bool ep, hipStream_t st) {
    d.tiles_m = (int)cdiv(d.M, 32 * plan.mb);
    d.tiles_k = (int)cdiv(d.K, DX_BK);
    d.splits = plan.splits;
    const mq_status s = nr == 1 ? launch_dx_nrs<1>(d, plan.mb, has8, ep, st) : nr == 2 ? launch_dx_nrs<2>(d, plan.mb, has8, ep, st)
                                                                                        : launch_dx_nrs<3>(d, plan.mb, has8, ep, st);
    if (s != MQ_OK || plan.splits == 1) return s;
    dx_finish_kernel<<<dim3((unsigned)(d.tiles_m * d.tiles_k * plan.mb * DX_RB * 4)), dim3(256), 0, st>>>(d, plan.mb);
    return launch_status();
}

}  // namespace mq
