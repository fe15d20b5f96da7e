// The fused forward for few tokens: K split over workgroups.
//
// A prompt or a calibration sample of M tokens gives the tiled forward kernel ceil(M / 160) * N / 128 workgroups: 32 of
// the 256 compute units for 77 tokens through a 4096 x 4096 layer, each walking all of K alone (35 us for 17 MB of codes).
// Here a workgroup takes one token tile of 32 .. 128 tokens, 128 channels and one range of K, runs the same main loop,
// and leaves its fp32 accumulators in the workspace in the order its lanes hold them (every store and load is a whole
// 1 KB line group); a second kernel adds the ranges in a fixed order and applies the forward's epilogue (and, with the
// objective or the gated unit, theirs).  The per-token sums of X that the epilogue needs come out of the tiles that pass
// through LDS anyway (block j of a tile is summed by the workgroups of channel tile j mod tiles_n), so the row-sum
// pre-pass and its launch disappear.
#include <algorithm>

#include "mq_linear.h"

namespace mq {

struct FwdRanges {
    float *part;     // [split][tile][bit-width][block of 16 channels][block of 16 tokens][256] four channels of one token each
    float *rs_part;  // [split][tiles_m * 32 MB] sums of X over the split's range of K
    int splits;
};
// The kernels' arguments: a launch costs by their bytes, and a kernel of a few microseconds by the lines that it reads of them.  With all of
// FwdArgs in both, and a branch on the counter at the end of the first, plain calls of one to three bit-widths took 1.1 to 1.6 % longer
// replayed from a graph, 2.7 to 3.5 % one after the other (235 sizes of up to 350 tokens).
struct FwdSplitArgs {  // (names as in FwdArgs)
    const uint16_t *X;
    const uint8_t *Q;
    int M, N, K;
    int r[3];
    int tiles_m, tiles_n;
    FwdRanges s;
    float *arrived;    // the counter of the finishing kernel, to be cleared
};
struct FwdPlainArgs {
    int M, N;
    int r[3];
    int tiles_m, tiles_n;
    const float *alpha, *zero;
    uint16_t *Y[3];
    int gate;
    uint16_t *A[3];
};
struct FwdLossArgs {
    int M, N;
    int r[3];
    int tiles_m, tiles_n;
    const float *alpha, *zero, *bias;
    uint16_t *Y[3];
    const uint16_t *T;
    uint16_t *dY[3];
    int teacher[3];
    float coef[3];
    int mix;
    float *partial;
    uint32_t *arrived;
    float *losses;
    int loss_slot[3];
    float inv_mn;
};
template <bool LOSS>
struct FwdFinishArgs {
    FwdRanges s;
    int mb;
    std::conditional_t<LOSS, FwdLossArgs, FwdPlainArgs> f;
};

template <int NR, bool HAS8, bool LAST2, bool EP, int MB>
__global__ __launch_bounds__(256, NR * MB <= 9 ? 2 : 1) void fwd_split_kernel(FwdSplitArgs a) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const FwdRanges &s = a.s;
    constexpr int BM = 32 * MB;
    const int tiles = a.tiles_m * a.tiles_n;
    // Neighbouring ids, which share an XCD's L2, are token tiles of one channel tile (the same codes), then channel tiles
    // of one K range (the same columns of X).
    const int lid = (int)xcd_contiguous_id(blockIdx.x, gridDim.x);
    const int split = lid / tiles, tile = lid % tiles;
    const int tn = tile / a.tiles_m, tm = tile % a.tiles_m;
    const int m0 = tm * BM, n0 = tn * FWD_BN;
    const int nkt = (a.K + BKT - 1) / BKT;
    const int kt0 = (int)((int64_t)nkt * split / s.splits), kt1 = (int)((int64_t)nkt * (split + 1) / s.splits);
    uint32_t rs_mask = 0;
    float rsum[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) {
        rsum[j] = 0.f;
        if (j % a.tiles_n == tn) rs_mask |= 1u << j;
    }
    f32x4 acc[NR][2][2 * MB];
    fwd_main_loop<NR, HAS8, LAST2, EP, MB, true>(a, smem, m0, n0, kt0, kt1 - kt0, min(a.K, kt1 * BKT), acc, rsum, rs_mask);

#pragma unroll
    for (int j = 0; j < MB; ++j)
        if (rs_mask & (1u << j)) {
            float v = rsum[j];
            v += __shfl_xor(v, 1, 64);
            v += __shfl_xor(v, 2, 64);
            v += __shfl_xor(v, 4, 64);
            // (the lanes beside clear the counter of the kernel that finishes, with the same store: at the head of this one 77 tokens, 4096 x
            // 4096 took 14.27 instead of 13.97 us)
            const bool sums = (threadIdx.x & 7) == 0;
            float *to = sums ? s.rs_part + (size_t)split * a.tiles_m * BM + m0 + j * 32 + (threadIdx.x >> 3) : a.arrived;
            if ((threadIdx.x & 7) < 2) *to = sums ? v : 0.f;
        }
    f32x4 *dst = reinterpret_cast<f32x4 *>(s.part) + ((size_t)split * tiles + tile) * (NR * MB * 4 * 256) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int tb = 0; tb < 2 * MB; ++tb)
                if (m0 + 16 * tb < a.M) dst[((i * 2 + rb) * 2 * MB + tb) * 256] = acc[i][rb][tb];
}

// Adds the K ranges and finishes the outputs.  Workgroup = (tile, 32 tokens, 32 channels): its waves take the four 16 x 16
// blocks and write 64 contiguous bytes of 32 tokens.  The arithmetic per output is that of the
// tiled forward kernel's epilogue.
template <int NR, bool LOSS>
__global__ __launch_bounds__(256) void fwd_split_finish_kernel(FwdFinishArgs<LOSS> p) {
    __shared__ float red[4][4];
    const auto &a = p.f;
    const FwdRanges &s = p.s;
    const int mb = p.mb;
    float *partial = nullptr;
    uint32_t *arrived = nullptr;
    if constexpr (LOSS) {  // (asked for at the end they are two more trips to memory)
        partial = a.partial;
        arrived = a.arrived;
        asm volatile("" : "+s"(partial), "+s"(arrived));
    }
    const int lane = threadIdx.x & 63, g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g4 = lane >> 4, l16 = lane & 15, rb = g & 1;
    const int w = blockIdx.x & 3, tb = (int)(blockIdx.x >> 2) % mb * 2 + (g >> 1), tile = (int)(blockIdx.x >> 2) / mb;
    const int tiles = a.tiles_m * a.tiles_n;
    const int tn = tile / a.tiles_m, tm = tile % a.tiles_m;
    const int m = tm * 32 * mb + tb * 16 + l16, n = tn * FWD_BN + w * 32 + rb * 16 + 4 * g4;
    const bool ok = m < a.M && n < a.N;

    const size_t rs_step = (size_t)a.tiles_m * 32 * mb, step = (size_t)tiles * NR * mb * 1024;
    const f32x4 *src = reinterpret_cast<const f32x4 *>(s.part) + (((size_t)tile * NR * 2 + rb) * 2 * mb + tb) * 256 + w * 64 + lane;
    f32x4 sum[NR];
    float rs = 0.f;
#pragma unroll
    for (int i = 0; i < NR; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int splits = tm * 32 * mb + tb * 16 < a.M ? s.splits : 0;  // (a block past the tokens has not been stored)
    // the loads of up to four ranges are in flight together (counted at compile time: a test around each load would be a branch)
    auto add = [&](auto count_tag, int p0) {
        constexpr int COUNT = decltype(count_tag)::value;
        f32x4 v[COUNT][NR];
        float r[COUNT];
#pragma unroll
        for (int p = 0; p < COUNT; ++p) {
            r[p] = s.rs_part[(p0 + p) * rs_step + m];
#pragma unroll
            for (int i = 0; i < NR; ++i) v[p][i] = __builtin_nontemporal_load(src + (p0 + p) * step + (size_t)i * mb * 1024);
        }
#pragma unroll
        for (int p = 0; p < COUNT; ++p) {
            rs += r[p];
#pragma unroll
            for (int i = 0; i < NR; ++i) sum[i] += v[p][i];
        }
    };
    int p0 = 0;
    for (; p0 + 4 <= splits; p0 += 4) add(std::integral_constant<int, 4>{}, p0);
    if (splits - p0 == 3) add(std::integral_constant<int, 3>{}, p0);
    if (splits - p0 == 2) add(std::integral_constant<int, 2>{}, p0);
    if (splits - p0 == 1) add(std::integral_constant<int, 1>{}, p0);

    u32x2 y[NR];
    float err[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) err[i] = 0.f;
    if (ok) {
        const f32x4 al = *reinterpret_cast<const f32x4 *>(a.alpha + n), ze = *reinterpret_cast<const f32x4 *>(a.zero + n);
        f32x4 bias = {0.f, 0.f, 0.f, 0.f};
        if constexpr (LOSS)
            if (a.bias) bias = *reinterpret_cast<const f32x4 *>(a.bias + n);
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const bool is8 = a.r[i] == 8;
            const float mult = is8 ? 1.0f : (float)(1 << (8 - a.r[i]));
            const float offset = is8 ? 0.0f : 128.0f * mult;
            float o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float t = (offset + ze[e]) * rs;
                const float inner = __builtin_fmaf(mult, sum[i][e], -t);
                o[e] = LOSS ? __builtin_fmaf(al[e], inner, bias[e]) : al[e] * inner;
            }
            y[i] = u32x2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
        }
        const size_t at = (size_t)m * a.N + n;
        u32x2 t = {0u, 0u};  // read before an output is written: a caller may let one take the target's place
        if constexpr (LOSS)
            if (a.T) t = *reinterpret_cast<const u32x2 *>(a.T + at);
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            if (a.Y[i]) *reinterpret_cast<u32x2 *>(a.Y[i] + at) = y[i];
            if constexpr (!LOSS)
                if (a.gate) {
                    auto gated = [&](uint32_t pair) {
                        const float gt = bf16_lo(pair), up = bf16_hi(pair);
                        return (a.gate == 2 ? silu(gt) : gelu_tanh(gt)) * up;
                    };
                    *reinterpret_cast<uint32_t *>(a.A[i] + (size_t)m * (a.N >> 1) + (n >> 1)) = pack_bf16x2(gated(y[i].x), gated(y[i].y));
                }
        }
        if constexpr (LOSS) {
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                u32x2 ref = t;
                const bool taught = a.teacher[i] >= 0;
#pragma unroll
                for (int u = 0; u < NR; ++u)
                    if (a.teacher[i] == u) ref = y[u];
                u32x2 o;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const float y0 = bf16_lo(y[i][c]), y1 = bf16_hi(y[i][c]);
                    float d0 = y0 - bf16_lo(ref[c]), d1 = y1 - bf16_hi(ref[c]);
                    if (a.mix && taught) {  // teacher and ground truth, weighted equally
                        const float e0 = y0 - bf16_lo(t[c]), e1 = y1 - bf16_hi(t[c]);
                        err[i] += 0.5f * (d0 * d0 + d1 * d1 + e0 * e0 + e1 * e1);
                        d0 = 0.5f * (d0 + e0);
                        d1 = 0.5f * (d1 + e1);
                    } else {
                        err[i] = __builtin_fmaf(d1, d1, __builtin_fmaf(d0, d0, err[i]));
                    }
                    o[c] = pack_bf16x2(a.coef[i] * d0, a.coef[i] * d1);
                }
                *reinterpret_cast<u32x2 *>(a.dY[i] + at) = o;
            }
        }
    }
    if constexpr (LOSS) {  // workgroup sums in a fixed order
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            float v = err[i];
#pragma unroll
            for (int msk = 1; msk < 64; msk <<= 1) v += __shfl_xor(v, msk, 64);
            if (lane == 0) red[g][i] = v;
        }
        __syncthreads();
        leave_sums<NR>(a, (int)threadIdx.x < NR ? red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x] : 0.f, tiles * mb * 4, partial, arrived);
    }
}

// ---- host side ------------------------------------------------------------------------------------
namespace {

template <int NR, bool HAS8, bool LAST2, bool EP, int MB>
mq_status launch_split_mb(const FwdSplitArgs &s, hipStream_t st) {
    if (!allow_lds<fwd_split_kernel<NR, HAS8, LAST2, EP, MB>>(split_lds(MB))) return MQ_ERR_DEVICE;
    fwd_split_kernel<NR, HAS8, LAST2, EP, MB><<<dim3(s.tiles_m * s.tiles_n * s.s.splits), dim3(256), split_lds(MB), st>>>(s);
    return launch_status();
}

template <int NR, bool HAS8, bool LAST2, bool EP>
mq_status launch_split_form(const FwdSplitArgs &s, int mb, hipStream_t st) {
    switch (mb) {
        case 1: return launch_split_mb<NR, HAS8, LAST2, EP, 1>(s, st);
        case 2: return launch_split_mb<NR, HAS8, LAST2, EP, 2>(s, st);
        case 3: return launch_split_mb<NR, HAS8, LAST2, EP, 3>(s, st);
    }
    if constexpr (split_mb(NR) == 4) return launch_split_mb<NR, HAS8, LAST2, EP, 4>(s, st);
    return MQ_ERR_SHAPE;  // (make_split_plan stays within split_mb)
}

template <int NR, bool HAS8, bool EP>
mq_status launch_split(const FwdSplitArgs &s, int mb, hipStream_t st) {
    // (one bit-width only: the look-up is a chain of dependent instructions, which low tiles at several bit-widths have nothing to put
    // between: 3440 x 1504, 20 tokens, r = 8/4/2 9.0 -> 9.6 us, 6288 x 3728, 60 tokens, 4/2 14.4 -> 15.0; 2512 x 3088, 213
    // tokens, r = 2 15.6 -> 14.5)
    if constexpr (NR == 1 && has_last2(NR, HAS8))
        if (s.r[NR - 1] == 2) return launch_split_form<NR, HAS8, true, EP>(s, mb, st);
    return launch_split_form<NR, HAS8, false, EP>(s, mb, st);
}

template <int NR>
mq_status launch_split_nr(const FwdSplitArgs &s, int mb, bool has8, bool ep, hipStream_t st) {
    if constexpr (NR == 1) ep = ep && !has8;  // the code of r = 8 is never rounded up past the byte
    if (has8) {
        if constexpr (NR > 1)
            if (ep) return launch_split<NR, true, true>(s, mb, st);
        return launch_split<NR, true, false>(s, mb, st);
    }
    return ep ? launch_split<NR, false, true>(s, mb, st) : launch_split<NR, false, false>(s, mb, st);
}

template <int NR>
mq_status launch_finish(const FwdRanges &s, const FwdArgs &f, int mb, bool loss, hipStream_t st, int64_t blocks) {
    if (loss) {
        const FwdLossArgs a{f.M, f.N, {f.r[0], f.r[1], f.r[2]}, f.tiles_m, f.tiles_n, f.alpha, f.zero, f.bias, {f.Y[0], f.Y[1], f.Y[2]}, f.T,
                            {f.dY[0], f.dY[1], f.dY[2]}, {f.teacher[0], f.teacher[1], f.teacher[2]}, {f.coef[0], f.coef[1], f.coef[2]}, f.mix,
                            f.partial, f.arrived, f.losses, {f.loss_slot[0], f.loss_slot[1], f.loss_slot[2]}, f.inv_mn};
        fwd_split_finish_kernel<NR, true><<<dim3((unsigned)blocks), dim3(256), 0, st>>>({s, mb, a});
    } else {
        const FwdPlainArgs a{f.M, f.N, {f.r[0], f.r[1], f.r[2]}, f.tiles_m, f.tiles_n, f.alpha, f.zero, {f.Y[0], f.Y[1], f.Y[2]}, f.gate, {f.A[0], f.A[1], f.A[2]}};
        fwd_split_finish_kernel<NR, false><<<dim3((unsigned)blocks), dim3(256), 0, st>>>({s, mb, a});
    }
    return launch_status();
}

}  // namespace

FwdSplitPlan fwd_split_plan(int64_t M, int64_t N, int64_t K, int nr) {
    return remembered<FwdSplitPlan>(make_split_plan, M, N, K, nr);
}

mq_status launch_fwd_split(const FwdArgs &f, const FwdSplitPlan &plan, int nr, bool has8, bool ep, bool loss, float *part, float *rs_part,
                           hipStream_t st, int64_t *blocks) {
    FwdArgs a = f;
    a.tiles_m = (int)cdiv(f.M, 32 * plan.mb);
    a.tiles_n = (int)cdiv(f.N, FWD_BN);
    *blocks = plan.loss_blocks;
    if (*blocks > kLossArrivals) a.arrived = nullptr;
    const FwdRanges ranges{part, rs_part, plan.splits};
    const FwdSplitArgs s{a.X, a.Q, a.M, a.N, a.K, {a.r[0], a.r[1], a.r[2]}, a.tiles_m, a.tiles_n, ranges, reinterpret_cast<float *>(f.arrived)};
    mq_status e = nr == 1 ? launch_split_nr<1>(s, plan.mb, has8, ep, st) : nr == 2 ? launch_split_nr<2>(s, plan.mb, has8, ep, st)
                                                                                    : launch_split_nr<3>(s, plan.mb, has8, ep, st);
    if (e != MQ_OK) return e;
    return nr == 1 ? launch_finish<1>(ranges, a, plan.mb, loss, st, *blocks) : nr == 2 ? launch_finish<2>(ranges, a, plan.mb, loss, st, *blocks)
                                                                                       : launch_finish<3>(ranges, a, plan.mb, loss, st, *blocks);
}

}  // namespace mq
