// mq_linear_fwd_multi / mq_linear_bwd: the nested quantized linear on the bf16 matrix cores.
//
// Forward (MatQuant objective, section 3.2: the same input goes through the layer once per
// bit-width): ONE pass over X and the int8 codes.  A workgroup (256 threads, one wave per SIMD) owns
// 128 output channels x 32 MB tokens (MB = 2 .. 6); four LDS stages of a [32 MB x 64] bf16 tile of X
// and a [128 x 64] tile of int8 codes are filled by direct global->LDS loads, every wave turns the
// codes of its 32 channels into one bf16 operand per requested bit-width in registers and issues
// 16x16x32 MFMAs into one accumulator set per bit-width.
//
//   r = 8     : int8 -> fp32 -> bf16 (exact, codes <= 255).
//   r < 8     : the slicing operator of section 3.2 on 16-bit lanes.  The byte is placed in the high
//               half of a 16-bit lane, a saturating add of half << 8 implements min(q + half, 255)
//               (the clamp of the slicing equation), a shift leaves the r-bit code, and OR-ing
//               0x4300 makes the bf16 number 128 + code.  The 128 is removed in the epilogue with
//               the per-token sum of X.  Extra precision (errata section) skips the saturation.
//
// Epilogue: Y = alpha_n * (2^s * acc - (2^s * 128 + z_n) * sum_k X[m,k]).
//
// Backward (identity STE): dX (mq_linear_wide.hip) reuses the in-register slicing on a transposed copy of the
// codes, with one pre-scaled gradient operand per bit-width accumulated into a single accumulator;
// dW is a plain bf16 GEMM of the lambda-weighted gradient sum against X.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "mq_linear.h"

namespace mq {

// ============================================================================================
// forward
// ============================================================================================
// row stride of the staging tile of the epilogue: the 8-byte writes of sixteen tokens and the 16-byte read-back spread over all banks
constexpr int FWD_OS = FWD_BN * 2 + 16;
static_assert(FWD_OS % 16 == 0, "rows of the staging tile are read in aligned pieces of 16 bytes");
constexpr int fwd_lds(int mb, int nr) {
    const int stages = FWD_STAGES * (mb * 32 * 128 + FWD_Q_TILE), staging = nr * mb * 32 * FWD_OS;
    return stages > staging ? stages : staging;
}

// One workgroup = 4 waves (one per SIMD, so each may use the whole 512-entry register file) on a
// (32 MB)-token x 128-channel tile; wave w owns channels [32 w, 32 w + 32) for all tokens, i.e.
// 4 MB NR accumulator blocks of 16 x 16.  A converted code operand (16 channels) is then reused by
// 2 MB MFMAs, which keeps the VALU slicing work at a fraction of the MFMA time.
// LDS holds four stages of 64 k: stage kt is computed while stage kt + 1 is resident (the operands
// of the next 32-wide k step are fetched into registers behind the MFMAs of the current one, also
// across the stage boundary) and stages kt + 2, kt + 3 are in flight, so a load has two full
// iterations to arrive.
//
// With three bit-widths and two or three token blocks, two workgroups fit a compute unit (at most 80 KB of LDS and 256
// registers each): one converts, stages and stores its outputs while the other multiplies.
template <int NR, bool HAS8, bool LAST2, bool EP, int MB, bool LOSS>
__global__ __launch_bounds__(256, MB <= 3 ? 2 : 1) void fwd_kernel(FwdArgs a) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    constexpr int BM = 32 * MB;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g4 = lane >> 4, l16 = lane & 15;

    // What the epilogue needs from the kernel arguments is fetched now, into scalar registers that stay
    // live through the main loop: read where it is used, each costs a scalar-memory round trip with
    // nothing to hide it (one wave per SIMD).
    const float *k_alpha = a.alpha, *k_zero = a.zero, *k_rowsum = a.rowsum, *k_bias = LOSS ? a.bias : nullptr;
    const uint16_t *k_T = LOSS ? a.T : nullptr;
    uint16_t *k_Y[NR], *k_dY[NR];
    float k_coef[NR];
    int k_teacher[NR], k_mix = LOSS ? a.mix : 0;
    uint16_t *k_A[NR];
    int k_gate = LOSS ? 0 : a.gate;
    asm volatile("" : "+s"(k_alpha), "+s"(k_zero), "+s"(k_rowsum));
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        k_Y[i] = a.Y[i];
        asm volatile("" : "+s"(k_Y[i]));
        k_A[i] = LOSS ? nullptr : a.A[i];
        if constexpr (!LOSS) asm volatile("" : "+s"(k_A[i]));
        if constexpr (LOSS) {
            k_dY[i] = a.dY[i];
            k_coef[i] = a.coef[i];
            k_teacher[i] = a.teacher[i];
            asm volatile("" : "+s"(k_dY[i]), "+s"(k_coef[i]), "+s"(k_teacher[i]));
        }
    }
    if constexpr (LOSS) asm volatile("" : "+s"(k_bias), "+s"(k_T), "+s"(k_mix));
    if constexpr (!LOSS) asm volatile("" : "+s"(k_gate));

    // XCD-aware tile order: each XCD walks groups of 4 token tiles across the channel tiles
    const uint32_t lid = xcd_contiguous_id(blockIdx.x, gridDim.x);
    constexpr int GROUP = 4;
    const int width = GROUP * a.tiles_n;
    const int first_m = (int)(lid / width) * GROUP;
    const int gsz = min(a.tiles_m - first_m, GROUP);
    const int tm = first_m + (int)(lid % width) % gsz;
    const int tn = (int)(lid % width) / gsz;
    const int m0 = tm * BM, n0 = tn * FWD_BN;

    f32x4 acc[NR][2][2 * MB];
    float no_rowsum[MB];
    fwd_main_loop<NR, HAS8, LAST2, EP, MB, false>(a, smem, m0, n0, 0, (a.K + BKT - 1) / BKT, a.K, acc, no_rowsum, 0u);

    // ---- epilogue ---------------------------------------------------------------------------
    // a lane holds channels 4 g4 .. 4 g4 + 3 of token l16 per 16 x 16 block.
    // It therefore owns only 4 consecutive channels of a token; the tile is first assembled in
    // LDS ([token][channel] bf16, FWD_OS) and then stored as whole 256-byte rows.
    constexpr int OS = FWD_OS;          // staging row stride in bytes
    constexpr int OT = BM * OS;         // one bit-width
    __syncthreads();                    // every wave is done with the operand stages
    float rs[2 * MB];
#pragma unroll
    for (int tb = 0; tb < 2 * MB; ++tb) {
        const int m = m0 + tb * 16 + l16;
        rs[tb] = m < a.M ? k_rowsum[m] : 0.f;
    }
    f32x4 alv[2], zev[2], bv[LOSS ? 2 : 1];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        const int nloc = wave * 32 + rb * 16 + 4 * g4;
        alv[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
        zev[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (LOSS) bv[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (n0 + nloc < a.N) {
            alv[rb] = *reinterpret_cast<const f32x4 *>(k_alpha + n0 + nloc);
            zev[rb] = *reinterpret_cast<const f32x4 *>(k_zero + n0 + nloc);
            if constexpr (LOSS)
                if (k_bias) bv[rb] = *reinterpret_cast<const f32x4 *>(k_bias + n0 + nloc);
        }
    }
    // LOSS: the lane's chunks of the target are requested now, behind the parameter loads, and
    // arrive while the accumulators are converted and staged.  With the largest accumulator sets
    // there are registers for some of them only; the others are requested after the staging and arrive
    // while the first ones are consumed.  (Nothing spills with these counts but at 96 tokens and three
    // bit-widths, whose two workgroups per compute unit leave 256 registers to a wave: three outside the
    // main loop, two of them without the objective too.)
    constexpr int CHUNKS = BM * 16 / 256;
    constexpr int EARLY = NR * MB > 12 || (NR == 3 && MB == 3) ? 2 : (NR * MB == 12 ? CHUNKS / 2 : CHUNKS);
    u32x4 tpre[LOSS ? CHUNKS : 1];
    auto request_target = [&](int it) {
        const int c = it * 256 + threadIdx.x;
        const int m = m0 + (c >> 4), n = n0 + (c & 15) * 8;
        tpre[it] = u32x4{0u, 0u, 0u, 0u};
        if (k_T && m < a.M && n < a.N)
            tpre[it] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(k_T + (size_t)m * a.N + n));
    };
    if constexpr (LOSS) {
#pragma unroll
        for (int it = 0; it < EARLY; ++it) request_target(it);
    }
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        const int nloc = wave * 32 + rb * 16 + 4 * g4;
        const f32x4 al = alv[rb], ze = zev[rb];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const bool is8 = HAS8 && i == 0;
            const float mult = is8 ? 1.0f : (float)(1 << (8 - a.r[i]));
            const float bias = is8 ? 0.0f : 128.0f * mult;
            float bz[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) bz[e] = bias + ze[e];
#pragma unroll
            for (int tb = 0; tb < 2 * MB; ++tb) {
                float y[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // (mult is a power of two, so the fused form rounds exactly like mult * acc - t)
                    const float t = bz[e] * rs[tb], v = acc[i][rb][tb][e];
                    const float inner = is8 ? v - t : __builtin_fmaf(mult, v, -t);
                    y[e] = LOSS ? __builtin_fmaf(al[e], inner, bv[rb][e]) : al[e] * inner;
                }
                const u32x2 o = {pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
                *reinterpret_cast<u32x2 *>(smem + i * OT + (tb * 16 + l16) * OS + nloc * 2) = o;
            }
        }
    }
    if constexpr (LOSS) {
#pragma unroll
        for (int it = EARLY; it < CHUNKS; ++it) request_target(it);
    }
    __syncthreads();
    if constexpr (!LOSS) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
#pragma unroll
            for (int it = 0; it < BM * 16 / 256; ++it) {
                const int c = it * 256 + threadIdx.x;
                const int row = c >> 4, ch = c & 15;
                const int m = m0 + row, n = n0 + ch * 8;
                if (m < a.M && n < a.N) {
                    const uint8_t *src = smem + i * OT + row * OS + ch * 16;
                    const u32x4 y = *reinterpret_cast<const u32x4 *>(src);
                    if (k_Y[i]) __builtin_nontemporal_store(y, reinterpret_cast<u32x4 *>(k_Y[i] + (size_t)m * a.N + n));
                    if (k_gate) {
                        // the gated unit on the rounded outputs, pair by pair (the arithmetic of mq_gated_unit_fwd)
                        const bool use_silu = k_gate == 2;
                        auto gated = [&](uint32_t pair) {
                            const float g = bf16_lo(pair), u = bf16_hi(pair);
                            return (use_silu ? silu(g) : gelu_tanh(g)) * u;
                        };
                        const u32x2 o = {pack_bf16x2(gated(y[0]), gated(y[1])), pack_bf16x2(gated(y[2]), gated(y[3]))};
                        __builtin_nontemporal_store(o, reinterpret_cast<u32x2 *>(k_A[i] + (size_t)m * (a.N >> 1) + (n >> 1)));
                    }
                }
            }
        }
    } else {
        // L2 objective on the staged tile (section 3.2 with the loss of section 3.1.2, co-distillation
        // targets of section 5.2): a lane takes the same 8 channels of a token from every bit-width
        // and from the target, adds (Y_i - T_i)^2 to its sums and stores dY_i = coef_i (Y_i - T_i);
        // the arithmetic per element is that of the stand-alone loss kernel, on the same rounded Y.
        float sum[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) sum[i] = 0.f;
        // The parameters of the objective are read once into vector registers (left to itself the compiler
        // reloads them from the kernel arguments for every chunk, a scalar-memory round trip each time):
        // the factor, the lane's addresses in dY_i / Y_i, and the choice of the teacher as bit masks.
        const int crow = threadIdx.x >> 4, cch = threadIdx.x & 15;  // chunk `it` is row crow + 16 it, channels 8 cch ..
        const size_t at0 = (size_t)(m0 + crow) * a.N + n0 + cch * 8;
        const bool cols_ok = n0 + cch * 8 < a.N;
        float cf[NR];
        uint32_t pick[NR][NR], mixed_slot[NR];
        uint16_t *pd[NR], *py[NR];
        int stored = 0, taught = 0;  // wave-uniform: bit i = Y_i is stored / slot i has a teacher
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            cf[i] = k_coef[i];
            pd[i] = k_dY[i] + at0;
            py[i] = k_Y[i] ? k_Y[i] + at0 : nullptr;
            stored |= k_Y[i] ? 1 << i : 0;
            taught |= k_teacher[i] >= 0 ? 1 << i : 0;
            mixed_slot[i] = k_teacher[i] >= 0 ? 0xFFFFFFFFu : 0u;
            asm volatile("" : "+v"(cf[i]), "+v"(pd[i]), "+v"(py[i]), "+v"(mixed_slot[i]));
#pragma unroll
            for (int u = 0; u < NR; ++u) {
                pick[i][u] = k_teacher[i] == u ? 0xFFFFFFFFu : 0u;
                asm volatile("" : "+v"(pick[i][u]));
            }
        }
        stored = __builtin_amdgcn_readfirstlane(stored);
        taught = __builtin_amdgcn_readfirstlane(taught);
        asm volatile("" : "+s"(stored), "+s"(taught));
        const size_t chunk_step = (size_t)16 * a.N;  // elements between a lane's consecutive chunks
        // The equal-weight mix of teacher and target, and the presence of any teacher at all, are variants
        // of the whole loop, chosen once: without teachers every bit-width is compared with the target and
        // the selection of the reference disappears.
        auto chunks = [&](auto mixed, auto teach) {
            constexpr bool MIX = decltype(mixed)::value, TEACH = decltype(teach)::value;
            // the staged values of chunk it + 1 are read (every chunk lies inside the tile) before chunk it is
            // worked on, outside the bounds test, so that the LDS latency hides behind arithmetic
            auto staged = [&](int it, u32x4 (&dst)[NR]) {
#pragma unroll
                for (int i = 0; i < NR; ++i) {
                    dst[i] = *reinterpret_cast<const u32x4 *>(smem + i * OT + (crow + 16 * it) * OS + cch * 16);
                }
            };
            u32x4 ynext[NR];
            staged(0, ynext);
#pragma unroll
            for (int it = 0; it < CHUNKS; ++it) {
                const int row = crow + 16 * it;
                u32x4 y[NR];
#pragma unroll
                for (int i = 0; i < NR; ++i) y[i] = ynext[i];
                if (it + 1 < CHUNKS) staged(it + 1, ynext);
                if (cols_ok && m0 + row < a.M) {
                    const u32x4 t = tpre[it];
#pragma unroll
                    for (int i = 0; i < NR; ++i) {
                        u32x4 tt = t;
                        if constexpr (TEACH) {
#pragma unroll
                            for (int u = 0; u < NR; ++u)
                                if (u != i) {
#pragma unroll
                                    for (int j = 0; j < 4; ++j) tt[j] = (y[u][j] & pick[i][u]) | (tt[j] & ~pick[i][u]);
                                }
                        }
                        u32x4 o;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float y0 = bf16_lo(y[i][j]), y1 = bf16_hi(y[i][j]);
                            float d0 = y0 - bf16_lo(tt[j]), d1 = y1 - bf16_hi(tt[j]);
                            if (MIX && mixed_slot[i]) {  // teacher and ground truth, weighted equally
                                const float e0 = y0 - bf16_lo(t[j]), e1 = y1 - bf16_hi(t[j]);
                                sum[i] += 0.5f * (d0 * d0 + d1 * d1 + e0 * e0 + e1 * e1);
                                d0 = 0.5f * (d0 + e0);
                                d1 = 0.5f * (d1 + e1);
                            } else {
                                sum[i] = __builtin_fmaf(d1, d1, __builtin_fmaf(d0, d0, sum[i]));
                            }
                            o[j] = pack_bf16x2(cf[i] * d0, cf[i] * d1);
                        }
                        __builtin_nontemporal_store(o, reinterpret_cast<u32x4 *>(pd[i] + it * chunk_step));
                        if (stored & (1 << i))
                            __builtin_nontemporal_store(y[i], reinterpret_cast<u32x4 *>(py[i] + it * chunk_step));
                    }
                }
            }
        };
        if (k_mix)
            chunks(std::true_type{}, std::true_type{});
        else if (taught)
            chunks(std::false_type{}, std::true_type{});
        else
            chunks(std::false_type{}, std::false_type{});
        // workgroup sums in a fixed order; the staging tiles are dead after the barrier
        __syncthreads();
        float *red = reinterpret_cast<float *>(smem);
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            float v = sum[i];
#pragma unroll
            for (int msk = 1; msk < 64; msk <<= 1) v += __shfl_xor(v, msk);
            if (lane == 0) red[wave * 4 + i] = v;
        }
        __syncthreads();
        float v = 0.f;
        if ((int)threadIdx.x < NR)
            for (int w = 0; w < 4; ++w) v += red[w * 4 + threadIdx.x];
        leave_sums<NR>(a, v, a.tiles_m * a.tiles_n, a.partial, a.arrived);
    }
}

// sum_k X[m, k] in fp32, one wave per row (and clears the counter of a forward with the objective, unless null)
__global__ __launch_bounds__(256) void rowsum_kernel(const uint16_t *__restrict__ X, int M, int K,
                                                     float *__restrict__ out, uint32_t *__restrict__ arrived) {
    if (arrived && blockIdx.x == 0 && threadIdx.x == 0) *arrived = 0u;
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (m >= M) return;
    const u32x4 *row = reinterpret_cast<const u32x4 *>(X + (size_t)m * K);
    float s = 0.f;
    for (int c0 = lane; c0 < K / 8; c0 += 256) {  // four loads in flight; the sum runs in the order of the chunks
        u32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = c0 + 64 * u < K / 8 ? row[c0 + 64 * u] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) s += __uint_as_float(v[u][i] << 16) + __uint_as_float(v[u][i] & 0xFFFF0000u);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) out[m] = s;
}

// ============================================================================================
// backward, preparation (HBM-bound): one pass over the nr gradient tensors produces
//   As_i[m, n] = bf16(lambda_i * alpha_n * 2^s_i * dY_i[m, n])     (operand of the dX contraction)
//   c[m]       = sum_i sum_n As_i[m, n] * (bias_i + z_n / 2^s_i)   (what the 128 + code form and z add to dX[m, :])
//   G[m, n]    = bf16(sum_i lambda_i * dY_i[m, n])                  (operand of the dW GEMM, turned or in pieces: dw_turns)
// ============================================================================================
struct PrepArgs {
    const uint16_t *dY[3];
    // GATED kernels: the layer is the stacked gate / up projection of a gated unit a = act(g) u and its output
    // gradients are formed here from GU_i [M, N] (columns (g, u) pairs) and dA_i [M, N / 2] instead of read from dY_i
    const uint16_t *GU[3];
    const uint16_t *dA[3];
    int silu;
    uint16_t *As[3];     // null pointers when dX is not wanted
    const float *alpha, *zero;
    float lam[3];
    float mult[3];       // 2^s_i
    float bias[3];       // 128 for sliced slots, 0 for the r = 8 slot
    float *cpart;        // [nsplit][M] partial sums of c over column ranges, or null
    uint16_t *G;         // the summed gradient in pieces of 32 tokens x 64 columns (summed_at), or null; zeros past M
    int turn;            // G is [M / 32][N][32] instead
    int nr, M, N;
    int cols_per_split;  // multiple of 64
    int strips, nsplit;  // token strips, column ranges
    // > 0: no sum; gradient i alone, times lam[i], goes to G + i * g_step (As and cpart are null, `each` times as many workgroups)
    int each;
    int64_t g_step;
    // the transposed copies that the same launch makes (null: not wanted): the codes for dX, the input for dW
    const uint8_t *Q;
    uint8_t *QT;         // [K, N]
    const uint16_t *X;
    uint16_t *XT;        // [M / 32][K][32], zeros past M
    int K;
};

constexpr int PREP_ROWS = 32;
constexpr int PREP_MAX_SPLIT = 16;

// Where G[m, n] is: [M / 32][N / 64][32][64], the last piece of columns as narrow as what is left of N.  A workgroup of dW reads 32
// tokens x 256 columns at a time, 16 KB in one place here.  From rows of N columns each they are 32 pieces far apart, and three lines
// instead of two where a row is no multiple of 128 bytes (18432 x 2304, 4096 tokens, both operands by rows 325 us, both in pieces 310).
__device__ __forceinline__ size_t summed_at(int m, int n, int N) {
    return ((size_t)(m >> 5) * N + (n & ~63)) * 32 + (m & 31) * min(64, N - (n & ~63)) + (n & 63);
}

// Workgroup (strip, split) walks 32 token rows across one range of columns in 32 x 64 tiles: thread
// (r, ch) = (t / 8, t % 8) owns eight consecutive columns of row r, so a row segment is one 128-byte
// line per gradient tensor.  Where the summed gradient is wanted turned, its tile goes through LDS and leaves as 64-byte row segments.
template <bool GATED>
__device__ __forceinline__ void prep_gradients(const PrepArgs &a, int strip, int split, uint16_t (*tile)[PREP_ROWS + 2]) {
    const int t = threadIdx.x, r = t >> 3, ch = t & 7;
    const int m0 = strip * PREP_ROWS, m = m0 + r;
    const int nbeg = split * a.cols_per_split, nend = min(nbeg + a.cols_per_split, a.N);
    const bool want_as = a.As[0] != nullptr;
    float c = 0.f;
    // what a tile reads; the loads of the next one are in flight while a tile is worked on and turned
    struct Raw {
        u32x4 v[3];
        u32x2 da[GATED ? 3 : 1];
    };
    auto load = [&](int n) {
        Raw x;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            x.v[i] = u32x4{0u, 0u, 0u, 0u};
            if constexpr (GATED) x.da[i] = u32x2{0u, 0u};
            if (i < a.nr && m < a.M && n < a.N) {
                if constexpr (GATED) {
                    x.v[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a.GU[i] + (size_t)m * a.N + n));
                    x.da[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(a.dA[i] + (size_t)m * (a.N >> 1) + (n >> 1)));
                } else {
                    x.v[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a.dY[i] + (size_t)m * a.N + n));
                }
            }
        }
        return x;
    };
    Raw next = load(nbeg + ch * 8);
    for (int n0 = nbeg; n0 < nend; n0 += 64) {
        const int n = n0 + ch * 8;
        const Raw raw = next;
        if (n0 + 64 < nend) next = load(n + 64);
        float g[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) g[j] = 0.f;
        if (m < a.M && n < a.N) {
            float al[8], ze[8];
            if (want_as) {
                *reinterpret_cast<f32x4 *>(al) = *reinterpret_cast<const f32x4 *>(a.alpha + n);
                *reinterpret_cast<f32x4 *>(al + 4) = *reinterpret_cast<const f32x4 *>(a.alpha + n + 4);
                *reinterpret_cast<f32x4 *>(ze) = *reinterpret_cast<const f32x4 *>(a.zero + n);
                *reinterpret_cast<f32x4 *>(ze + 4) = *reinterpret_cast<const f32x4 *>(a.zero + n + 4);
            }
            u32x4 dy[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                if (i >= a.nr) break;
                dy[i] = raw.v[i];
                if constexpr (GATED) {
                    // the gradient of the gated unit, pair by pair, rounded to bf16 like mq_gated_unit_bwd does
                    const u32x2 da = raw.da[i];
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        dy[i][w] = gated_pair_grad(bf16_lo(raw.v[i][w]), bf16_hi(raw.v[i][w]),
                                                   (w & 1) ? bf16_hi(da[w >> 1]) : bf16_lo(da[w >> 1]), a.silu != 0);
                }
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                if (i >= a.nr) break;
                const float f = a.lam[i] * a.mult[i], inv = 1.0f / a.mult[i];
                u32x4 o;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float dlo = bf16_bits_to_float(dy[i][w] & 0xFFFFu), dhi = bf16_bits_to_float(dy[i][w] >> 16);
                    g[2 * w] += a.lam[i] * dlo;
                    g[2 * w + 1] += a.lam[i] * dhi;
                    if (want_as) {
                        o[w] = pack_bf16x2(dlo * (f * al[2 * w]), dhi * (f * al[2 * w + 1]));
                        c += bf16_bits_to_float(o[w] & 0xFFFFu) * (a.bias[i] + ze[2 * w] * inv);
                        c += bf16_bits_to_float(o[w] >> 16) * (a.bias[i] + ze[2 * w + 1] * inv);
                    }
                }
                if (want_as) *reinterpret_cast<u32x4 *>(a.As[i] + (size_t)m * a.N + n) = o;
            }
        }
        if (a.turn) {
            __syncthreads();  // the previous tile has been written out
#pragma unroll
            for (int j = 0; j < 8; ++j) tile[ch * 8 + j][r] = (uint16_t)float_to_bf16_bits(g[j]);
            __syncthreads();
            const int nn = t >> 2, part = t & 3;  // 64 columns, four 16-byte pieces each
            if (n0 + nn < a.N) {
                const uint32_t *src = reinterpret_cast<const uint32_t *>(&tile[nn][part * 8]);
                *reinterpret_cast<u32x4 *>(a.G + ((size_t)strip * a.N + n0 + nn) * 32 + part * 8) =
                    u32x4{src[0], src[1], src[2], src[3]};
            }
        } else if (a.G && n < a.N)
            *reinterpret_cast<u32x4 *>(a.G + summed_at(m, n, a.N)) =
                u32x4{pack_bf16x2(g[0], g[1]), pack_bf16x2(g[2], g[3]), pack_bf16x2(g[4], g[5]), pack_bf16x2(g[6], g[7])};
    }
    if (a.cpart) {
        c += __shfl_xor(c, 1, 64);
        c += __shfl_xor(c, 2, 64);
        c += __shfl_xor(c, 4, 64);
        if (ch == 0 && m < a.M) a.cpart[(size_t)split * a.M + m] = c;
    }
}

// Transposed copies.  Whole 128-byte lines are read, 16 bytes per lane; the elements of neighbouring rows are first put side
// by side in registers, so that the LDS tile is written in dwords (a byte or a 16-bit value at a time, the LDS writes were
// what took the time), and leave as 16-byte pieces.

// 128 x 128 codes: QT[k][n] = Q[n][k].  Thread (g, ch) turns rows 4 g .. 4 g + 3, columns 16 ch .. 16 ch + 15.  The tile holds
// 128 rows of 128 bytes, 144 bytes apart; the 16-byte pieces of row c are at positions piece ^ (c / 16), which spreads a wave's
// dword writes over the banks.
constexpr int QT_STRIDE = 36;  // dwords
__device__ __forceinline__ void transpose_codes(const PrepArgs &a, int tn, int tk, uint32_t *tile) {
    const int t = threadIdx.x, n0 = tn * 128, k0 = tk * 128;
    {
        const int g = t >> 3, ch = t & 7;
        u32x4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = n0 + 4 * g + i, k = k0 + 16 * ch;  // (N, K are multiples of 16)
            v[i] = n < a.N && k < a.K ? __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a.Q + (size_t)n * a.K + k)) : u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            // bytes of four rows -> dwords of four columns
            const uint32_t lo01 = __builtin_amdgcn_perm(v[1][w], v[0][w], 0x05010400u), hi01 = __builtin_amdgcn_perm(v[1][w], v[0][w], 0x07030602u);
            const uint32_t lo23 = __builtin_amdgcn_perm(v[3][w], v[2][w], 0x05010400u), hi23 = __builtin_amdgcn_perm(v[3][w], v[2][w], 0x07030602u);
            const uint32_t col[4] = {__builtin_amdgcn_perm(lo23, lo01, 0x05040100u), __builtin_amdgcn_perm(lo23, lo01, 0x07060302u),
                                     __builtin_amdgcn_perm(hi23, hi01, 0x05040100u), __builtin_amdgcn_perm(hi23, hi01, 0x07060302u)};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                tile[(16 * ch + 4 * w + j) * QT_STRIDE + (((g >> 2) ^ ch) << 2) + (g & 3)] = col[j];
        }
    }
    __syncthreads();
    const int piece = t & 7;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = (t >> 3) + 32 * i, k = k0 + c, n = n0 + 16 * piece;
        if (k < a.K && n < a.N)
            *reinterpret_cast<u32x4 *>(a.QT + (size_t)k * a.N + n) =
                *reinterpret_cast<const u32x4 *>(tile + c * QT_STRIDE + ((piece ^ (c >> 4)) << 2));
    }
}

// 64 tokens x 64 columns of X into the token blocks of dw_kernel's operand: element (m, k) goes to
// ((m / 32) K + k) 32 + m % 32.  Thread (g, ch) turns tokens 2 g, 2 g + 1 of columns 8 ch .. 8 ch + 7.  A column of a token
// block is 16 dwords, 20 apart, with 8 more after every eight columns: a wave's dword writes touch every bank once.
__device__ __forceinline__ int xt_at(int block, int col) { return block * (8 * 168) + (col >> 3) * 168 + (col & 7) * 20; }
constexpr int XT_TILE = 2 * 8 * 168;  // dwords
__device__ __forceinline__ void transpose_input(const PrepArgs &a, int tm, int tk, uint32_t *tile) {
    const int t = threadIdx.x, m0 = tm * 64, k0 = tk * 64;
    {
        const int g = t >> 3, ch = t & 7;
        u32x4 v[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int m = m0 + 2 * g + i, k = k0 + 8 * ch;
            v[i] = m < a.M && k < a.K ? __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a.X + (size_t)m * a.K + k)) : u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            tile[xt_at(g >> 4, 8 * ch + 2 * w) + (g & 15)] = __builtin_amdgcn_perm(v[1][w], v[0][w], 0x05040100u);
            tile[xt_at(g >> 4, 8 * ch + 2 * w + 1) + (g & 15)] = __builtin_amdgcn_perm(v[1][w], v[0][w], 0x07060302u);
        }
    }
    __syncthreads();
    const int piece = t & 3, k = k0 + (t >> 2);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int m = m0 + 32 * b + 8 * piece;
        if (k < a.K && (m & ~31) < a.M)
            *reinterpret_cast<u32x4 *>(a.XT + ((size_t)(m >> 5) * a.K + k) * 32 + (m & 31)) =
                *reinterpret_cast<const u32x4 *>(tile + xt_at(b, t >> 2) + 4 * piece);
    }
}

// The whole preparation of a backward in one launch: the first strips x nsplit workgroups take the gradients, then come the
// tiles of Q and of X that have to be turned.  (As three launches in a row, each a few microseconds for a small layer and
// each with a tail in which most compute units wait: 16 x 256 x 256 10.8 us, 400 x 3600 x 3600 28 us.)
template <bool GATED>
__global__ __launch_bounds__(256) void bwd_prep_kernel(PrepArgs a) {
    __shared__ __attribute__((aligned(16))) uint32_t smem[128 * QT_STRIDE];
    static_assert(XT_TILE <= 128 * QT_STRIDE && 64 * (PREP_ROWS + 2) * 2 <= 128 * QT_STRIDE * 4, "tiles share the LDS");
    int b = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    const int gradients = a.strips * a.nsplit;
    if (b < gradients * max(a.each, 1)) {
        if (a.each) {
            const int i = b / gradients;
            a.dY[0] = i == 0 ? a.dY[0] : i == 1 ? a.dY[1] : a.dY[2];
            a.lam[0] = i == 0 ? a.lam[0] : i == 1 ? a.lam[1] : a.lam[2];
            a.G += i * a.g_step;
            a.nr = 1;
            b %= gradients;
        }
        prep_gradients<GATED>(a, b % a.strips, b / a.strips, reinterpret_cast<uint16_t(*)[PREP_ROWS + 2]>(smem));
        return;
    }
    b -= gradients * max(a.each, 1);
    const int qk = (a.K + 127) >> 7, codes = a.QT ? qk * ((a.N + 127) >> 7) : 0;
    if (b < codes) {
        transpose_codes(a, b / qk, b % qk, smem);
        return;
    }
    b -= codes;
    const int xk = (a.K + 63) >> 6, inputs = a.XT ? xk * ((a.M + 63) >> 6) : 0;
    if (b >= inputs) return;
    transpose_input(a, b / xk, b % xk, smem);
}

// ============================================================================================
// backward dW: dW[n, k] (+)= sum_m G[m, n] * X[m, k]   (plain bf16 GEMM, fp32 out)
// ============================================================================================
struct DwArgs {
    // TURN: the operand of each gradient is [M, N] as the caller has it, or in pieces (summed_at), X is [M, K].  Otherwise both come
    // turned, in blocks of 32 tokens, [M / 32][rows][32]: the 64-byte row segments that one LDS stage takes from a tile's 256 rows
    // are then one contiguous 16 KB piece of memory, i.e. whole 128-byte lines.
    const uint16_t *G[3];
    const uint16_t *X;
    int in_pieces;
    float *dW;             // [N, K] per gradient
    float *part;           // [split tiles][parts][side][side]: partial tiles of the tiles that are cut
    int M, N, K;
    int accumulate;
    int tiles_n, tiles_k;
    int whole;             // work items [0, whole) are whole tiles; the others are token ranges of the remaining tiles
    int parts;             // token ranges per remaining tile
};  // (several gradients against the same X: tile t belongs to gradient t / (tiles_n tiles_k))

static DwPlan dw_plan(int64_t M, int64_t N, int64_t K, int batch) { return remembered<DwPlan>(make_dw_plan, M, N, K, batch); }

// Same pipeline as the forward and dX kernels (one wave per SIMD, direct-to-LDS stages, operand work fenced in between the
// MFMAs), without any code conversion.  The four
// waves form a 2 x 2 grid over the tile.  HB = 4, a 256 x 256 tile, 128 x 128 per wave: 64 accumulators of 16 x 16 (all 256
// accumulator registers), 16 operand reads per 64 MFMAs - the square wave tile is what keeps the LDS traffic (32 KB read + 16 KB
// written per 16 tokens and compute unit, 94 bytes per clock at the matrix-core rate) under the 128 bytes per clock the LDS
// delivers.  HB = 2, a 128 x 128 tile, 64 x 64 per wave: 16 accumulators, 8 reads per 16 MFMAs, two workgroups to a compute
// unit.  Stages are one 32-token step deep; five of them fill the LDS (HB = 2: half of it).
//
// TURN: the contraction index (tokens) runs across the rows of both operands, as the caller left them, and the LDS turns them on the
// way to the registers (ds_read_b64_tr_b16: four tokens of sixteen columns at a time), so that no transposed copies are
// written and read back.  See dw_turns for what it costs and where it is used.
template <int HB, bool TURN>
__global__ __launch_bounds__(256) void dw_kernel(DwArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    constexpr int RB = 2 * HB, NM = RB * RB;         // 16-row blocks of either operand per wave, MFMAs per stage
    constexpr int DW_BN = dw_side(HB), DW_BK = dw_side(HB);
    constexpr int DW_A_TILE = DW_BN * 64, DW_STAGE = DW_A_TILE + DW_BK * 64;
    constexpr int AL = DW_BN / 64, BL = DW_BK / 64;  // direct-to-LDS loads per wave and stage (16 rows each)
    constexpr int LPS = AL + BL;
    static_assert(LPS <= NM / 2, "not enough MFMAs to hide the loads");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave >> 1, wk = wave & 1;
    const int g4 = lane >> 4, l16 = lane & 15;

    // work item -> tile and token range
    const int nmt_all = (a.M + DW_BM - 1) / DW_BM;
    uint32_t lid;
    int mt0 = 0, mt1 = nmt_all;
    float *dst = nullptr;
    bool to_part = false;
    if ((int)blockIdx.x < a.whole) {
        lid = xcd_contiguous_id(blockIdx.x, (uint32_t)a.whole);
    } else {
        const int idx = (int)blockIdx.x - a.whole, part = idx % a.parts;
        lid = (uint32_t)(a.whole + idx / a.parts);
        mt0 = (int)((int64_t)nmt_all * part / a.parts);
        mt1 = (int)((int64_t)nmt_all * (part + 1) / a.parts);
        dst = a.part + (size_t)idx * (DW_BN * DW_BK);
        to_part = true;
    }
    const uint32_t tiles = (uint32_t)(a.tiles_n * a.tiles_k);
    const uint32_t grad = lid / tiles;
    lid %= tiles;
    const uint16_t *G = grad == 0 ? a.G[0] : grad == 1 ? a.G[1] : a.G[2];
    if (!to_part) dst = a.dW + (size_t)grad * a.N * a.K;
    constexpr int GROUP = 4;
    const int width = GROUP * a.tiles_k;
    const int first_n = (int)(lid / width) * GROUP;
    const int gsz = min(a.tiles_n - first_n, GROUP);
    const int tn = first_n + (int)(lid % width) % gsz;
    const int tk = (int)(lid % width) / gsz;
    const int n0 = tn * DW_BN, k0 = tk * DW_BK;

    // TURN: LDS layout of an operand's stage: pieces of 8 tokens x 64 columns (1 KB, what one load instruction of a wave writes), piece
    // (token group g, column group c) at (g + 4 c) KB; inside, eight rows of 128 bytes, in which the block of columns 16 p .. is at
    // position p ^ (row / 2 % 2) ^ 2 (g % 2).  A transposing read takes 32 bytes of four rows for each group of sixteen lanes, lane
    // group g those of token group g: those of neighbouring groups then fall on all 64 banks.
    // Wave w loads token group w, instruction i column group i, eight neighbouring lanes a whole 128-byte line of a row (two pieces
    // of 64 bytes, apart in the wave: 8 % longer).
    const int lpos = ((lane >> 1) & 3) ^ ((lane >> 4) & 1) ^ (2 * (wave & 1));
    const int lrow = 8 * wave + (lane >> 3), lcol = lpos * 16 + (lane & 1) * 8;
    uint32_t goff[AL], xoff[BL];   // byte offsets inside a stage of 32 tokens, out of range for columns past the operand's end
    if constexpr (TURN) {
#pragma unroll
        for (int i = 0; i < AL; ++i) {
            const int row = a.in_pieces ? min(64, a.N - n0 - 64 * i) : a.N;   // elements of a row
            goff[i] = n0 + lcol + 64 * i < a.N ? (uint32_t)(lrow * row + lcol + (a.in_pieces ? 2048 : 64) * i) * 2u : kOOB;
        }
#pragma unroll
        for (int i = 0; i < BL; ++i) xoff[i] = k0 + lcol + 64 * i < a.K ? (uint32_t)(lrow * a.K + lcol + 64 * i) * 2u : kOOB;
    } else {
        uint32_t off0;
        int col;
        u8_tile_lane<4>(wave, lane, 0, 64u, off0, col);   // 64 rows of 64 bytes per instruction
#pragma unroll
        for (int i = 0; i < AL; ++i) goff[i] = off0 + i * 4096u;
#pragma unroll
        for (int i = 0; i < BL; ++i) xoff[i] = off0 + i * 4096u;
    }
    const bool g_blocks = !TURN || a.in_pieces;   // 32 tokens of N elements each are one block of memory

    // The descriptors of a stage start at the tile's first column in the first of its 32 tokens and end with the last token of the range
    // (or of M; a block of memory, which has zeros past M, with the block), so what is past it is out of range and answered with zeros
    // without touching memory: the loads in flight are the same every stage.  Stages are requested in their order: the bases walk along.
    const uint16_t *g_base = G + (size_t)mt0 * DW_BM * a.N + (size_t)n0 * (g_blocks ? DW_BM : 1);
    const uint16_t *x_base = a.X + (size_t)mt0 * DW_BM * a.K + (size_t)k0 * (TURN ? 1 : DW_BM);
    const size_t g_block = (size_t)a.N * DW_BM, x_block = (size_t)a.K * DW_BM;
    int rows_left = min(a.M, mt1 * DW_BM) - mt0 * DW_BM;   // from the stage that is requested next
    u32x4 g_rsrc, x_rsrc;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr)(smem) + wave * 1024);
    auto next_stage = [&] {
        // (31 rows of 2^22 columns and a tile are less than 2^31 bytes)
        const int rows = min(max(rows_left, 0), DW_BM);
        g_rsrc = scalar_rsrc(g_base, g_blocks ? (rows > 0 ? a.N - n0 : 0) * (2 * DW_BM) : max(rows * a.N - n0, 0) * 2);
        x_rsrc = scalar_rsrc(x_base, TURN ? max(rows * a.K - k0, 0) * 2 : (rows > 0 ? a.K - k0 : 0) * (2 * DW_BM));
        g_base += g_block;
        x_base += x_block;
        rows_left -= DW_BM;
    };
    // Load l of that stage into LDS buffer `buf` as the compiler's own load, for the small tiles of copies: it deals the scalar instructions of a
    // stage over the products.  With all of them at the start of a stage, where nothing else runs (or in pieces behind the products of its second half),
    // dW calls of 768 tokens and more take 1.02 times as long, of fewer 1.007 (560 sizes); 256-tiles 0.993.
    constexpr bool COMPILED = HB == 2 && !TURN;
    auto compiled_load = [&](auto l_tag, int buf) {
        constexpr int l = decltype(l_tag)::value;
        const int bytes = rows_left > 0 ? (l < AL ? a.N - n0 : a.K - k0) * (2 * DW_BM) : 0;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(l < AL ? g_base : x_base, bytes),
                                                 (lds_ptr)(smem + buf * DW_STAGE + wave * 1024 + (l < AL ? l * 4096 : DW_A_TILE + (l - AL) * 4096)), 16,
                                                 l < AL ? goff[l < AL ? l : 0] : xoff[l < AL ? 0 : l - AL], 0, 0, 0);
        if (l == LPS - 1) {
            g_base += g_block;
            x_base += x_block;
            rows_left -= DW_BM;
        }
    };
    // LDS fragment offsets inside a stage (TURN: by the block of 16 columns in its group of 64): lane (l16, g4) ends up with eight
    // tokens of column l16 of a block, those of group g4 (otherwise of its chunk of a row of 32)
    uint32_t gb[TURN ? 4 : 1], xb[TURN ? 4 : 1];
    if constexpr (TURN) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const uint32_t at = (uint32_t)(g4 * 1024 + (l16 >> 2) * 128 + ((p ^ (l16 >> 3) ^ (2 * (g4 & 1))) << 5) + (l16 & 3) * 8);
            gb[p] = at + (uint32_t)(wn * (RB / 4) * 4096);
            xb[p] = at + (uint32_t)(DW_A_TILE + wk * (RB / 4) * 4096);
        }
    } else {
        const uint32_t at = (uint32_t)(l16 * 64) + ((uint32_t)(group_chunk(g4) ^ ((l16 >> 2) & 3)) << 4);
        gb[0] = at + (uint32_t)(wn * RB * 1024);
        xb[0] = at + (uint32_t)(DW_A_TILE + wk * RB * 1024);
    }
    auto read_half = [&](u32x4 &dst, const uint8_t *stage, const auto &at, auto block_tag, auto half_tag) {
        constexpr int B = decltype(block_tag)::value, HALF = decltype(half_tag)::value;
        if constexpr (TURN) {
            const u32x2 v = read_turned16(stage + at[B & 3] + (B >> 2) * 4096 + HALF * 512);
            dst[2 * HALF] = v[0];
            dst[2 * HALF + 1] = v[1];
        } else if constexpr (HALF == 0) {   // (one read brings both)
            dst = *reinterpret_cast<const u32x4 *>(stage + at[0] + B * 1024);
        }
    };
    constexpr std::integral_constant<int, 0> first{};
    constexpr std::integral_constant<int, 1> second{};

    f32x4 acc[RB][RB];   // [block of n][block of k]: rows 4 g4 .. 4 g4 + 3, column l16 of the block
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < RB; ++j) acc[rb][j] = f32x4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
    for (int st = 0; st < DW_NST - 1; ++st) {
        if constexpr (COMPILED) {
            static_for<LPS>([&](auto l) { compiled_load(l, st); });
        } else {
            next_stage();
#pragma unroll
            for (int i = 0; i < LPS; ++i)
                load_to_lds(i < AL ? g_rsrc : x_rsrc, i < AL ? goff[i] : xoff[i - AL], lds0 + st * DW_STAGE + (i < AL ? i * 4096 : DW_A_TILE + (i - AL) * 4096));
        }
    }
    stage_barrier<(DW_NST - 2) * LPS, 0>();

    // The products of a stage come in two halves, over the first and over the second half of the columns' blocks.  Every operand
    // has one register: the second half of the columns is read in the first half of the stage, the first half of the columns and
    // each block of rows, as soon as it is done with, are read for the next stage in the second half.
    u32x4 gf[RB], xf[RB];
    static_for<RB>([&](auto rb) {
        read_half(gf[decltype(rb)::value], smem, gb, rb, first);
        read_half(gf[decltype(rb)::value], smem, gb, rb, second);
    });
    static_for<RB / 2>([&](auto j) {
        read_half(xf[decltype(j)::value], smem, xb, j, first);
        read_half(xf[decltype(j)::value], smem, xb, j, second);
    });

    // one stage; cb = LDS buffer of this stage
    // (MORE = false, the last stage of the small tiles: nothing to prepare)
    auto tile = [&](int cb, auto more_tag) {
        constexpr bool MORE = decltype(more_tag)::value;
        const int nb = cb + 1 == DW_NST ? 0 : cb + 1;   // buffer of the next stage
        const int ib = cb == 0 ? DW_NST - 1 : cb - 1;   // buffer of the stage NST - 1 further on (= the one of the stage before)
        const uint8_t *cur = smem + cb * DW_STAGE, *nxt = smem + nb * DW_STAGE;
        [[maybe_unused]] const uint32_t fill = lds0 + ib * DW_STAGE;
        // products from one load to the next; instructions between the descriptors and the first load that reads one: products, reads, aim
        constexpr int EVERY = NM / 2 / LPS, READS = std::min(EVERY, RB), BETWEEN = EVERY + (TURN ? READS : (READS + 1) / 2) + 1;
        static_assert(COMPILED || BETWEEN >= kDescriptorWait, "wait states between a descriptor and the load that reads it");
        if constexpr (MORE && !COMPILED) next_stage();
        __builtin_amdgcn_sched_barrier(0);
        static_for<NM>([&](auto q_tag) {
            constexpr int q = decltype(q_tag)::value, H = NM / 2, HJ = RB / 2;
            constexpr int half = q / H, rb = q % H / HJ, j = half * HJ + q % HJ;
            mfma16_acc<HB == 4>(acc[rb][j], gf[rb], xf[j]);
            // one read, and one instruction of a load, behind a product
            if constexpr (half == 0) {
                if constexpr (q < 2 * HJ) read_half(xf[HJ + q / 2], cur, xb, std::integral_constant<int, HJ + q / 2>{}, std::integral_constant<int, q % 2>{});
                constexpr int l = q / EVERY;
                static_assert(EVERY >= 2 && H % LPS == 0, "a product between the two pieces of a load");
                if constexpr (MORE && COMPILED && q % EVERY == EVERY - 1) compiled_load(std::integral_constant<int, l>{}, ib);
                if constexpr (MORE && !COMPILED && q % EVERY == EVERY - 2) aim_load_to_lds<l < AL ? l * 4096 : DW_A_TILE + (l - AL) * 4096>(fill);
                if constexpr (MORE && !COMPILED && q % EVERY == EVERY - 1) aimed_load_to_lds(l < AL ? g_rsrc : x_rsrc, l < AL ? goff[l < AL ? l : 0] : xoff[l < AL ? 0 : l - AL]);
            } else if constexpr (MORE) {
                constexpr int p = q - H;
                if constexpr (p < 2 * HJ) read_half(xf[p / 2], nxt, xb, std::integral_constant<int, p / 2>{}, std::integral_constant<int, p % 2>{});
                if constexpr (p % HJ == 0 && p > 0) read_half(gf[rb - 1], nxt, gb, std::integral_constant<int, rb - 1>{}, second);
                if constexpr (p % HJ == HJ - 1) read_half(gf[rb], nxt, gb, std::integral_constant<int, rb>{}, first);
                if constexpr (p == H - 1) read_half(gf[rb], nxt, gb, std::integral_constant<int, rb>{}, second);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        mfma16_settle();
    };

    // The small tiles have a copy of the code for the last stage, which does not wait for one that nobody multiplies: with few
    // tokens there is no other (4096 x 4096, 19 tokens 20.6 -> 19.6 us).  With 256 accumulator registers the copy is not worth its
    // moves (fwd_main_loop).
    constexpr bool APART = HB == 2;
    int cb = 0;
    for (int mt = mt0; mt < mt1 - (APART ? 1 : 0); ++mt) {
        // Stage mt + 1 must be resident (operands read for it inside this stage); the loads of stages mt + 2 and mt + 3 may stay
        // in flight; after the barrier the buffer of stage mt - 1, all of whose operands have been multiplied, is free for stage
        // mt + 4.
        // (a counter of reads in flight ends at 15)
        stage_barrier<(DW_NST - 3) * LPS, std::min(15, (TURN ? 2 : 1) * (RB + RB / 2))>();
        tile(cb, std::true_type{});
        cb = cb + 1 == DW_NST ? 0 : cb + 1;
    }
    if constexpr (APART) tile(cb, std::false_type{});
    wait_vm0();  // loads of stages that nobody consumes must have landed before the workgroup ends

    // Two neighbouring column blocks exchange half of their lanes, after which a store instruction writes 32 consecutive k (one
    // 128-byte line) of two rows (lines left to two instructions of 64 bytes per row: 9216 x 2304, 16 tokens 17.2 -> 21.7 us).
    // Branch-free: every store goes through a buffer descriptor that starts at the first
    // element of the wave's 16-row block and ends with the destination, so rows past N fall out of range and are
    // dropped by the memory unit; a column past K is sent out of range explicitly.  The row part of the
    // address (wave-uniform) travels in the scalar offset, the lane part in one register per pair of blocks.
    // A token range of a cut tile writes its whole partial tile instead (row length = side of the tile, no edges).
    // When accumulating, the old values of a row block are requested together, one memory round trip for all of them.
    const int ld = to_part ? DW_BK : a.K;              // row length of the destination
    const int rows = to_part ? DW_BN : a.N - n0;       // rows and columns of the destination from this tile's origin
    const int cols = to_part ? DW_BK : a.K - k0;
    float *origin = to_part ? dst : dst + (int64_t)n0 * a.K + k0;
    uint32_t voff[RB / 2];
#pragma unroll
    for (int jp = 0; jp < RB / 2; ++jp) {
        const int c = wk * 16 * RB + jp * 32 + (lane & 31);
        voff[jp] = c < cols ? ((uint32_t)(8 * (lane >> 5)) * (uint32_t)ld + (uint32_t)c) * 4u : kOOB;
    }
    auto store_tile = [&](auto accumulate_tag) {
        constexpr bool ACCUMULATE = decltype(accumulate_tag)::value;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int r0 = wn * 16 * RB + rb * 16;                      // first row of the block inside the tile
            const int64_t left = ((int64_t)rows - r0) * ld - (to_part ? 0 : k0);  // elements to the end of the destination
            const __amdgpu_buffer_rsrc_t rW = make_rsrc(origin + (int64_t)r0 * ld, left > 0 ? (uint64_t)left * 4u : 0u);
            uint32_t old[ACCUMULATE ? 8 : 1][RB / 2];
            if constexpr (ACCUMULATE) {
#pragma unroll
                for (int row = 0; row < 8; ++row)
#pragma unroll
                    for (int jp = 0; jp < RB / 2; ++jp)
                        old[row][jp] = __builtin_amdgcn_raw_buffer_load_b32(rW, voff[jp], (uint32_t)row * (uint32_t)ld * 4u, 0);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int jp = 0; jp < RB / 2; ++jp) {
                    // rows (0 and 8) + e in the first result, (4 and 12) + e in the second
                    const auto two = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[rb][2 * jp][e]), __float_as_uint(acc[rb][2 * jp + 1][e]),
                                                                      false, false);
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int row = 4 * u + e;
                        float v = __uint_as_float(two[u]);
                        if constexpr (ACCUMULATE) v = __uint_as_float(old[row][jp]) + v;
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rW, voff[jp], (uint32_t)row * (uint32_t)ld * 4u, 0);
                    }
                }
        }
    };
    if (a.accumulate && !to_part)
        store_tile(std::true_type{});
    else
        store_tile(std::false_type{});
#else
    (void)a;
#endif
}

// dW tile (+)= the partial tiles of its token ranges, added in the order of the ranges.  A thread takes four rows of four
// columns, a workgroup 64 / HB rows of a split tile.
template <int HB>
__global__ __launch_bounds__(256) void dw_reduce_kernel(DwArgs a) {
    constexpr int SIDE = dw_side(HB), ROWS = 64 / HB, TPR = SIDE / 4;
    const int t = blockIdx.x / (SIDE / ROWS), rblock = blockIdx.x % (SIDE / ROWS);   // split tile, row block
    uint32_t lid = (uint32_t)(a.whole + t);
    const uint32_t tiles = (uint32_t)(a.tiles_n * a.tiles_k);
    float *dW = a.dW + (size_t)(lid / tiles) * a.N * a.K;
    lid %= tiles;
    constexpr int GROUP = 4;
    const int width = GROUP * a.tiles_k;
    const int first_n = (int)(lid / width) * GROUP;
    const int gsz = min(a.tiles_n - first_n, GROUP);
    const int tn = first_n + (int)(lid % width) % gsz;
    const int tk = (int)(lid % width) / gsz;
    const int row = rblock * ROWS + (threadIdx.x / TPR) * 4, col = (threadIdx.x % TPR) * 4;
    const int k = tk * SIDE + col;
    if (k >= a.K) return;   // (K is a multiple of 8: four columns are inside or outside together)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
        const int n = tn * SIDE + row + rr;
        if (n >= a.N) return;
        const float *src = a.part + (size_t)t * a.parts * (SIDE * SIDE) + (size_t)(row + rr) * SIDE + col;
        f32x4 sum = *reinterpret_cast<const f32x4 *>(src);
        for (int p = 1; p < a.parts; ++p) sum += *reinterpret_cast<const f32x4 *>(src + (size_t)p * (SIDE * SIDE));
        f32x4 *out = reinterpret_cast<f32x4 *>(dW + (size_t)n * a.K + k);
        if (a.accumulate) sum += *out;
        *out = sum;
    }
}

// ============================================================================================
// host side
// ============================================================================================

struct BwdWorkspace {
    size_t cvec, as[3], g, qt, xt, dwp, dxp, total;
};

static BwdWorkspace bwd_layout(int64_t M, int64_t N, int64_t K, int nr, const DxPlan &dx, const DwPlan &dw) {
    BwdWorkspace w;
    size_t o = 0;
    w.cvec = o;
    o += align256((size_t)PREP_MAX_SPLIT * M * 4);
    for (int i = 0; i < 3; ++i) {
        w.as[i] = o;
        if (i < nr) o += align256((size_t)M * N * 2);
    }
    const size_t m32 = ((size_t)M + 31) & ~(size_t)31;   // the operands of dW come in blocks of 32 tokens
    w.g = o;
    o += align256(m32 * N * 2);
    w.qt = o;
    o += align256((size_t)N * K);
    w.xt = o;
    o += align256(m32 * K * 2);
    // one of dX and dW is done before the other begins: their partial sums share their place
    w.dxp = w.dwp = o;
    o += align256(std::max(dw.part_bytes, dx.part_bytes));
    w.total = o;
    return w;
}
static BwdWorkspace bwd_layout(int64_t M, int64_t N, int64_t K, int nr) {
    return bwd_layout(M, N, K, nr, dx_plan(M, N, K, nr), dw_plan(M, N, K, 1));
}

static mq_status check_rs(const int *rs, int nr) {
    if (!rs) return MQ_ERR_NULL;
    if (nr < 1 || nr > 3) return MQ_ERR_BITS;
    for (int i = 0; i < nr; ++i) {
        if (rs[i] < 1 || rs[i] > 8) return MQ_ERR_BITS;
        for (int j = 0; j < i; ++j)
            if (rs[j] == rs[i]) return MQ_ERR_BITS;
    }
    return MQ_OK;
}

template <int HB, bool TURN>
static mq_status launch_dw_side(const DwArgs &w, const DwPlan &plan, hipStream_t st) {
    if (!allow_lds<dw_kernel<HB, TURN>>(dw_lds(HB))) return MQ_ERR_DEVICE;
    dw_kernel<HB, TURN><<<dim3(plan.whole + plan.rest * plan.parts), dim3(256), dw_lds(HB), st>>>(w);
    if (plan.rest > 0) dw_reduce_kernel<HB><<<dim3(plan.rest * HB * HB), dim3(256), 0, st>>>(w);
    return launch_status();
}

static mq_status launch_dw(DwArgs w, const DwPlan &plan, bool turn, hipStream_t st) {
    w.tiles_n = plan.tiles_n;
    w.tiles_k = plan.tiles_k;
    w.whole = plan.whole;
    w.parts = plan.parts;
    if (turn) return plan.hb == 2 ? launch_dw_side<2, true>(w, plan, st) : launch_dw_side<4, true>(w, plan, st);
    return plan.hb == 2 ? launch_dw_side<2, false>(w, plan, st) : launch_dw_side<4, false>(w, plan, st);
}

template <int NR, bool HAS8, bool LAST2, bool EP, int MB, bool LOSS>
static mq_status launch_fwd_mb(FwdArgs a, hipStream_t st, int64_t *blocks) {
    a.tiles_m = (int)cdiv(a.M, 32 * MB);
    a.tiles_n = (int)cdiv(a.N, FWD_BN);
    *blocks = (int64_t)a.tiles_m * a.tiles_n;
    if (*blocks > kLossArrivals) a.arrived = nullptr;
    if (!allow_lds<fwd_kernel<NR, HAS8, LAST2, EP, MB, LOSS>>(fwd_lds(MB, NR))) return MQ_ERR_DEVICE;
    fwd_kernel<NR, HAS8, LAST2, EP, MB, LOSS><<<dim3(a.tiles_m * a.tiles_n), dim3(256), fwd_lds(MB, NR), st>>>(a);
    return launch_status();
}

template <int NR, bool HAS8, bool LAST2, bool EP, bool LOSS>
static mq_status launch_fwd(const FwdArgs &a, hipStream_t st, int64_t *blocks) {
    constexpr int HI = fwd_mb(NR), LO = HI - 1;
    int mb = HI;
    fwd_tiled_cost(a.M, a.N, a.K, NR, &mb);
    if constexpr (NR == 3) {
        if (mb == 2) return launch_fwd_mb<NR, HAS8, LAST2, EP, 2, LOSS>(a, st, blocks);
        if (mb == 3) return launch_fwd_mb<NR, HAS8, LAST2, EP, 3, LOSS>(a, st, blocks);
    }
    return mb == LO ? launch_fwd_mb<NR, HAS8, LAST2, EP, LO, LOSS>(a, st, blocks) : launch_fwd_mb<NR, HAS8, LAST2, EP, HI, LOSS>(a, st, blocks);
}

template <int NR, bool HAS8, bool LOSS>
static mq_status launch_fwd_ep(const FwdArgs &a, bool ep, hipStream_t st, int64_t *blocks) {
    if constexpr (has_last2(NR, HAS8))
        if (a.r[NR - 1] == 2) return ep ? launch_fwd<NR, HAS8, true, true, LOSS>(a, st, blocks) : launch_fwd<NR, HAS8, true, false, LOSS>(a, st, blocks);
    return ep ? launch_fwd<NR, HAS8, false, true, LOSS>(a, st, blocks) : launch_fwd<NR, HAS8, false, false, LOSS>(a, st, blocks);
}

template <bool LOSS>
static mq_status launch_fwd_any(const FwdArgs &a, int nr, bool has8, bool ep, hipStream_t st, int64_t *blocks) {
    if (nr == 1)
        return has8 ? launch_fwd_ep<1, true, LOSS>(a, ep, st, blocks) : launch_fwd_ep<1, false, LOSS>(a, ep, st, blocks);
    if (nr == 2)
        return has8 ? launch_fwd_ep<2, true, LOSS>(a, ep, st, blocks) : launch_fwd_ep<2, false, LOSS>(a, ep, st, blocks);
    return has8 ? launch_fwd_ep<3, true, LOSS>(a, ep, st, blocks) : launch_fwd_ep<3, false, LOSS>(a, ep, st, blocks);
}

// Workspace of the forward: the tiled kernel's row sums at offset 0, the objective's partial sums (a bound over both
// forms: the tiled kernel at its smallest token tile, 64 tokens, or the finishing kernel of the split form) and the
// counter that goes with them, and what the split form keeps.
struct FwdWorkspace {
    size_t loss, counter, rs_part, part, total;
};
static FwdWorkspace fwd_layout(int64_t M, int64_t N, const FwdSplitPlan &plan, bool loss) {
    FwdWorkspace w;
    w.loss = align256((size_t)M * 4);
    const int64_t blocks = std::max<int64_t>(cdiv(M, 64) * cdiv(N, FWD_BN), plan.mb ? plan.loss_blocks : 0);
    w.counter = w.loss + (loss ? (size_t)blocks * 16 : 0);
    w.rs_part = align256(w.counter + 256);
    w.part = w.rs_part + (plan.mb ? align256(plan.rs_bytes) : 0);
    w.total = plan.mb ? w.part + plan.part_bytes : w.counter + 256;
    return w;
}

}  // namespace mq

extern "C" size_t mq_workspace_bytes(int op, int64_t M, int64_t N, int64_t K, int nr) {
    using namespace mq;
    if (op == MQ_OP_GEMV)  // M = B, nr = bits per code
        return M < 1 || M > 16 || N < 0 || K < 1 || nr < 1 || nr > 8 ? 0 : std::max<size_t>(256, gemv_split_workspace_bytes(M, N, K, nr));
    if (M < 0 || N < 0 || K < 0 || nr < 1 || nr > 3) return 0;
    if (op == MQ_OP_LINEAR_FWD || op == MQ_OP_LINEAR_FWD_L2)
        return fwd_layout(M, N, fwd_split_plan(M, N, K, nr), op == MQ_OP_LINEAR_FWD_L2).total;
    if (op == MQ_OP_LINEAR_BWD) return bwd_layout(M, N, K, nr).total + 256;
    if (op == MQ_OP_FFN_DECODE) return ffn_workspace_bytes(M, N, K);
    if (op == MQ_OP_L2_LOSS) return loss_workspace_bytes(M, N);
    if (op == MQ_OP_LINEAR_BWD_CLIP) return clip_workspace_bytes(M, N, K, nr);
    if (op == MQ_OP_AFFINE_BWD) return affine_workspace_bytes(M, N, K);
    return 0;
}

namespace mq {

// the L2 objective evaluated in the forward epilogue (user order; mapped to slots below)
struct FwdLoss {
    const uint16_t *target;
    const int *teacher;
    const float *lambda;
    uint16_t *const *dY;
    float *losses;
    uint32_t mix;
    const float *bias;
};

static mq_status fwd_run(const uint16_t *X, const uint8_t *Q, const float *alpha, const float *zero, int64_t M,
                         int64_t N, int64_t K, const int *rs, int nr, uint32_t flags, uint16_t *const *Y,
                         const FwdLoss *loss, void *ws, size_t ws_bytes, void *hip_stream,
                         bool check_only = false, uint16_t *const *gated_out = nullptr, int gate = 0,
                         bool tiled_only = false) {
    if (M < 0 || N < 0 || K < 1) return MQ_ERR_SHAPE;
    if (M > 0x7FFFFF00 || N > 0x7FFFFF00 || K > (1 << 22)) return MQ_ERR_SHAPE;
    if (cdiv(M, 128) * cdiv(N, FWD_BN) > 0x7FFFFFFF) return MQ_ERR_SHAPE;  // tiles of one launch (lower ones are taken only where theirs fit, too)
    mq_status s = check_rs(rs, nr);
    if (s != MQ_OK) return s;
    if (K % 16 != 0 || N % 8 != 0) return MQ_ERR_ALIGN;
    bool need_target = false;
    if (loss) {
        need_target = loss->mix || !loss->teacher;
        if (loss->teacher)
            for (int i = 0; i < nr; ++i) {
                if (loss->teacher[i] < -1 || loss->teacher[i] >= nr || loss->teacher[i] == i) return MQ_ERR_SHAPE;
                if (loss->teacher[i] < 0) need_target = true;
            }
    }
    if (M == 0 || N == 0) return MQ_OK;
    if (!X || !Q || !alpha || !zero) return MQ_ERR_NULL;
    if (!loss && !Y && !gate) return MQ_ERR_NULL;
    if (gate && !gated_out) return MQ_ERR_NULL;
    for (int i = 0; i < nr; ++i) {
        uint16_t *yi = Y ? Y[i] : nullptr;
        if (!loss && !gate && !yi) return MQ_ERR_NULL;
        if (yi && !aligned16(yi)) return MQ_ERR_ALIGN;
        if (gate && !gated_out[i]) return MQ_ERR_NULL;
        if (gate && (reinterpret_cast<uintptr_t>(gated_out[i]) & 7u)) return MQ_ERR_ALIGN;
    }
    if (loss) {
        if (!loss->dY || !loss->losses || (need_target && !loss->target)) return MQ_ERR_NULL;
        for (int i = 0; i < nr; ++i) {
            if (!loss->dY[i]) return MQ_ERR_NULL;
            if (!aligned16(loss->dY[i])) return MQ_ERR_ALIGN;
        }
        if (loss->target && !aligned16(loss->target)) return MQ_ERR_ALIGN;
        if (loss->bias && !aligned16(loss->bias)) return MQ_ERR_ALIGN;
    }
    if (!aligned16(X) || !aligned16(Q) || !aligned16(alpha) || !aligned16(zero)) return MQ_ERR_ALIGN;
    if (check_only) return MQ_OK;  // every argument but the workspace is fine
    FwdSplitPlan plan = tiled_only ? FwdSplitPlan{} : fwd_split_plan(M, N, K, nr);
    FwdWorkspace lay = fwd_layout(M, N, plan, loss != nullptr);
    if (plan.mb && ws_bytes < lay.total) {
        // a workspace that was made for more tokens, where K is not cut, still serves fewer
        plan = FwdSplitPlan{};
        lay = fwd_layout(M, N, plan, loss != nullptr);
    }
    if (!ws || ws_bytes < lay.total || !aligned16(ws)) return MQ_ERR_WORKSPACE;
    uint8_t *base = static_cast<uint8_t *>(ws);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);

    FwdArgs a{};
    a.X = X;
    a.Q = Q;
    a.alpha = alpha;
    a.zero = zero;
    a.rowsum = static_cast<float *>(ws);
    a.M = (int)M;
    a.N = (int)N;
    a.K = (int)K;
    // slot order: the r = 8 slot (if any) first
    int has8 = 0, pos = 0;
    int slot_of[3] = {0, 0, 0};
    for (int i = 0; i < 3; ++i) {
        a.Y[i] = nullptr;
        a.A[i] = nullptr;
        a.r[i] = 8;
    }
    a.gate = gate;
    for (int i = 0; i < nr; ++i)
        if (rs[i] == 8) {
            has8 = 1;
            slot_of[i] = 0;
        }
    pos = has8;
    for (int i = 0; i < nr; ++i)
        if (rs[i] != 8) slot_of[i] = pos++;
    for (int i = 0; i < nr; ++i) {
        a.Y[slot_of[i]] = Y ? Y[i] : nullptr;
        a.A[slot_of[i]] = gate ? gated_out[i] : nullptr;
        a.r[slot_of[i]] = rs[i];
    }
    a.arrived = reinterpret_cast<uint32_t *>(base + lay.counter);
    const double mn = (double)M * (double)N;
    if (loss) {
        a.T = loss->target;
        a.bias = loss->bias;
        a.mix = loss->mix ? 1 : 0;
        a.partial = reinterpret_cast<float *>(base + lay.loss);
        a.losses = loss->losses;
        a.inv_mn = (float)(1.0 / mn);
        for (int i = 0; i < nr; ++i) {
            const int sl = slot_of[i];
            a.loss_slot[i] = sl;
            a.dY[sl] = loss->dY[i];
            const int th = loss->teacher ? loss->teacher[i] : -1;
            a.teacher[sl] = th < 0 ? -1 : slot_of[th];
            a.coef[sl] = (float)((loss->lambda ? (double)loss->lambda[i] : 1.0) * 2.0 / mn);
        }
    }

    const bool ep = flags & MQ_FLAG_EXTRA_PRECISION;
    int64_t blocks = 0;
    if (plan.mb) {
        s = launch_fwd_split(a, plan, nr, has8, ep, loss != nullptr, reinterpret_cast<float *>(base + lay.part),
                             reinterpret_cast<float *>(base + lay.rs_part), st, &blocks);
    } else {
        rowsum_kernel<<<dim3((unsigned)cdiv(M, 4)), dim3(256), 0, st>>>(X, (int)M, (int)K, static_cast<float *>(ws), loss ? a.arrived : nullptr);
        const int wide = nr == 1 && !loss ? fwd_wide_mb(M, N, K, nullptr) : 0;
        s = wide ? launch_fwd_wide(a, wide, has8, ep, st)
            : loss ? launch_fwd_any<true>(a, nr, has8, ep, st, &blocks) : launch_fwd_any<false>(a, nr, has8, ep, st, &blocks);
    }
    if (s != MQ_OK || !loss || blocks <= kLossArrivals) return s;
    return launch_loss_finish(a.partial, blocks, nr, a.inv_mn, loss->losses, st, slot_of);
}

// 16-byte chunks of zeros (a kernel, not a memset node: callers may capture the stream into a graph)
__global__ __launch_bounds__(256) void zero_fill_kernel(u32x4 *__restrict__ dst, int64_t chunks) {
    for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < chunks; c += (int64_t)gridDim.x * 256)
        dst[c] = u32x4{0u, 0u, 0u, 0u};
}

}  // namespace mq

extern "C" mq_status mq_linear_fwd_multi(const uint16_t *X, const uint8_t *Q, const float *alpha,
                                         const float *zero, int64_t M, int64_t N, int64_t K, const int *rs,
                                         int nr, uint32_t flags, uint16_t *const *Y, void *ws, size_t ws_bytes,
                                         void *hip_stream) {
    return mq::fwd_run(X, Q, alpha, zero, M, N, K, rs, nr, flags, Y, nullptr, ws, ws_bytes, hip_stream);
}

extern "C" mq_status mq_linear_fwd_multi_gated(const uint16_t *X, const uint8_t *Q, const float *alpha,
                                               const float *zero, int64_t M, int64_t F, int64_t K, const int *rs,
                                               int nr, uint32_t flags, uint16_t *const *GU, uint16_t *const *A,
                                               void *ws, size_t ws_bytes, void *hip_stream) {
    if (F < 0 || F > 0x3FFFFF00) return MQ_ERR_SHAPE;
    if (F % 4 != 0) return MQ_ERR_ALIGN;  // rows of A start on 8-byte boundaries
    return mq::fwd_run(X, Q, alpha, zero, M, 2 * F, K, rs, nr, flags, GU, nullptr, ws, ws_bytes, hip_stream, false, A,
                       (flags & MQ_FLAG_FFN_SILU) ? 2 : 1);
}

// ---- the forward for callers that cannot allocate --------------------------------------------------
// Scratch of mq_linear_fwd_multi_noalloc: the per-token sums of X that the forward's pre-pass writes and
// its epilogue reads, in device memory that belongs to the library image (one copy per GPU, held until
// the process ends) instead of a caller workspace.
namespace mq {
constexpr int64_t kNoAllocMaxTokens = 1 << 18;
constexpr int kNoAllocMaxDevices = 64;
static __device__ __align__(256) float scratch[kNoAllocMaxTokens + 64];
// device address of `scratch` per GPU (the array's name is only a host-side handle), looked up once per device
static void *g_scratch_addr[kNoAllocMaxDevices];
static std::mutex g_scratch_mutex;

static mq_status noalloc_scratch(void **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kNoAllocMaxDevices) return MQ_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_addr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return MQ_ERR_DEVICE;
        g_scratch_addr[dev] = ptr;
    }
    *out = g_scratch_addr[dev];
    return MQ_OK;
}
}  // namespace mq

extern "C" mq_status mq_linear_fwd_multi_noalloc(const uint16_t *X, const uint8_t *Q, const float *alpha,
                                                 const float *zero, int64_t M, int64_t N, int64_t K, const int *rs,
                                                 int nr, uint32_t flags, uint16_t *const *Y, void *hip_stream) {
    using namespace mq;
    if (M > kNoAllocMaxTokens) return MQ_ERR_SHAPE;  // more tokens than the built-in scratch holds
    // the arguments are checked before the device is touched; an empty call launches nothing and needs no scratch
    mq_status s = fwd_run(X, Q, alpha, zero, M, N, K, rs, nr, flags, Y, nullptr, nullptr, 0, hip_stream, true);
    if (s != MQ_OK || M == 0 || N == 0) return s;
    void *ws = nullptr;
    s = noalloc_scratch(&ws);
    if (s != MQ_OK) return s;
    return fwd_run(X, Q, alpha, zero, M, N, K, rs, nr, flags, Y, nullptr, ws, sizeof(float) * (kNoAllocMaxTokens + 64),
                   hip_stream, false, nullptr, 0, true);
}

extern "C" mq_status mq_linear_fwd_multi_l2(const uint16_t *X, const uint8_t *Q, const float *alpha,
                                            const float *zero, int64_t M, int64_t N, int64_t K, const int *rs,
                                            int nr, uint32_t flags, const float *bias, const uint16_t *target,
                                            const int *teacher, const float *lambda, uint16_t *const *Y,
                                            uint16_t *const *dY, float *losses, void *ws, size_t ws_bytes,
                                            void *hip_stream) {
    const mq::FwdLoss loss{target, teacher, lambda, dY, losses, flags & MQ_FLAG_LOSS_MIX, bias};
    return mq::fwd_run(X, Q, alpha, zero, M, N, K, rs, nr, flags, Y, &loss, ws, ws_bytes, hip_stream);
}

namespace mq {
// fills in the cut of the gradients and launches the preparation
static mq_status launch_prep(PrepArgs &p, bool gated, hipStream_t st) {
    // column ranges so that about a thousand workgroups exist; c[m] is summed over them in the dX epilogue
    const int64_t M = p.M, N = p.N, K = p.K, strips = cdiv(M, PREP_ROWS);
    const int nsplit = (int)std::min<int64_t>(std::min<int64_t>(PREP_MAX_SPLIT, cdiv(N, 64)), std::max<int64_t>(1, cdiv(1024, strips)));
    p.cols_per_split = (int)(cdiv(cdiv(N, nsplit), 64) * 64);
    p.strips = (int)strips;
    p.nsplit = (int)cdiv(N, p.cols_per_split);
    const int64_t blocks = strips * p.nsplit * std::max(p.each, 1) + (p.QT ? cdiv(N, 128) * cdiv(K, 128) : 0) + (p.XT ? cdiv(M, 64) * cdiv(K, 64) : 0);
    if (blocks > 0x7F000000) return MQ_ERR_SHAPE;
    const int64_t gx = std::min<int64_t>(blocks, 1 << 20);
    const dim3 grid((unsigned)gx, (unsigned)cdiv(blocks, gx));
    if (gated)
        bwd_prep_kernel<true><<<grid, dim3(256), 0, st>>>(p);
    else
        bwd_prep_kernel<false><<<grid, dim3(256), 0, st>>>(p);
    return launch_status();
}

// Workspace of dw_each: the gradients and X, turned or scaled, and the partial tiles
struct EachWorkspace {
    size_t g_step, xt, dwp, total;  // g_step in bytes
};
static EachWorkspace each_layout(int64_t M, int64_t N, int64_t K, int nr, const DwPlan &dw) {
    EachWorkspace w;
    const size_t m32 = ((size_t)M + 31) & ~(size_t)31;
    w.g_step = align256(m32 * N * 2);
    w.xt = w.g_step * nr;
    w.dwp = w.xt + align256(m32 * K * 2);
    w.total = w.dwp + align256(dw.part_bytes);
    return w;
}

size_t dw_each_bytes(int64_t M, int64_t N, int64_t K, int nr, bool least) {
    return each_layout(M, N, K, nr, least ? dw_plan_whole(N, K, nr) : dw_plan(M, N, K, nr)).total;
}

// (no argument checks: the caller has made those of mq_linear_bwd)
mq_status dw_each(const uint16_t *X, const uint16_t *const *dY, const float *lambda, int64_t M, int64_t N, int64_t K, int nr,
                  float *out, uint8_t *ws, size_t ws_bytes, hipStream_t st) {
    DwPlan cut = dw_plan(M, N, K, nr);
    if (ws_bytes < each_layout(M, N, K, nr, cut).total) cut = dw_plan_whole(N, K, nr);
    const EachWorkspace lay = each_layout(M, N, K, nr, cut);
    DwArgs w{};
    bool scaled = false;
    for (int i = 0; i < nr; ++i) {
        scaled = scaled || (lambda && lambda[i] != 1.0f);
        w.G[i] = dY[i];
    }
    const bool turn = dw_turns(M, N, K, nr, !scaled, scaled, cut.hb);
    w.in_pieces = scaled;
    w.X = X;
    if (scaled || !turn) {  // otherwise the operands are taken as they stand
        PrepArgs p{};
        for (int i = 0; i < nr; ++i) {
            p.dY[i] = dY[i];
            p.lam[i] = lambda ? lambda[i] : 1.0f;
            w.G[i] = reinterpret_cast<uint16_t *>(ws + i * lay.g_step);
        }
        for (int i = 0; i < 3; ++i) p.mult[i] = 1.0f;
        p.G = reinterpret_cast<uint16_t *>(ws);
        p.turn = !turn;
        p.g_step = (int64_t)(lay.g_step / 2);
        p.each = p.nr = nr;
        p.M = (int)M;
        p.N = (int)N;
        p.K = (int)K;
        if (!turn) {
            p.X = X;
            w.X = p.XT = reinterpret_cast<uint16_t *>(ws + lay.xt);
        }
        const mq_status s = launch_prep(p, false, st);
        if (s != MQ_OK) return s;
    }
    w.dW = out;
    w.part = reinterpret_cast<float *>(ws + lay.dwp);
    w.M = (int)M;
    w.N = (int)N;
    w.K = (int)K;
    return launch_dw(w, cut, turn, st);
}

// gated: the output gradients come from GU and dA (see PrepArgs) instead of dY
static mq_status bwd_run(bool gated, const uint16_t *X, const uint8_t *Q, const float *alpha, const float *zero,
                         const uint16_t *const *dY, const uint16_t *const *GU, const uint16_t *const *dA,
                         const float *lambda, int64_t M, int64_t N, int64_t K, const int *rs, int nr, uint32_t flags,
                         uint16_t *dX, float *dW, void *ws, size_t ws_bytes, void *hip_stream) {
    if (M < 0 || N < 0 || K < 1) return MQ_ERR_SHAPE;
    if (M > (1 << 22) || N > (1 << 22) || K > (1 << 22)) return MQ_ERR_SHAPE;
    mq_status s = check_rs(rs, nr);
    if (s != MQ_OK) return s;
    if (K % 16 != 0 || N % 16 != 0) return MQ_ERR_ALIGN;
    if (M == 0 || N == 0) {
        // empty sums: dW (over no tokens) and dX (over no channels) are zero
        hipStream_t st0 = static_cast<hipStream_t>(hip_stream);
        const bool zero_dw = M == 0 && N > 0 && dW && !(flags & MQ_FLAG_ACCUM_DW), zero_dx = N == 0 && M > 0 && dX;
        if (!zero_dw && !zero_dx) return MQ_OK;
        if (M == 0 && N > 0 && dW && !(flags & MQ_FLAG_ACCUM_DW)) {
            if (!aligned16(dW)) return MQ_ERR_ALIGN;
            zero_fill_kernel<<<dim3((unsigned)std::min<int64_t>(cdiv(N * K / 4, 256), 65536)), dim3(256), 0, st0>>>(
                reinterpret_cast<u32x4 *>(dW), N * K / 4);
        }
        if (N == 0 && M > 0 && dX) {
            if (!aligned16(dX)) return MQ_ERR_ALIGN;
            zero_fill_kernel<<<dim3((unsigned)std::min<int64_t>(cdiv(M * K / 8, 256), 65536)), dim3(256), 0, st0>>>(
                reinterpret_cast<u32x4 *>(dX), M * K / 8);
        }
        return launch_status();
    }
    if (gated) {
        if (!GU || !dA) return MQ_ERR_NULL;
        for (int i = 0; i < nr; ++i) {
            if (!GU[i] || !dA[i]) return MQ_ERR_NULL;
            if (!aligned16(GU[i]) || !aligned16(dA[i])) return MQ_ERR_ALIGN;
        }
    } else {
        if (!dY) return MQ_ERR_NULL;
        for (int i = 0; i < nr; ++i) {
            if (!dY[i]) return MQ_ERR_NULL;
            if (!aligned16(dY[i])) return MQ_ERR_ALIGN;
        }
    }
    if (dX && (!Q || !alpha || !zero)) return MQ_ERR_NULL;
    if (dW && !X) return MQ_ERR_NULL;
    if ((dX && !aligned16(dX)) || (dW && !aligned16(dW)) || (X && !aligned16(X)) || (Q && !aligned16(Q)) ||
        (alpha && !aligned16(alpha)) || (zero && !aligned16(zero)))
        return MQ_ERR_ALIGN;
    // (a workspace that was made for more tokens may be too small for the partial sums of fewer: then nothing is cut)
    DxPlan dx_cut = dx_plan(M, N, K, nr);
    DwPlan dw_cut = dw_plan(M, N, K, 1);
    BwdWorkspace lay = bwd_layout(M, N, K, nr, dx_cut, dw_cut);
    if (ws_bytes < lay.total + 256) {
        if (dx_cut.part_bytes) dx_cut = DxPlan{5, 1, 0};
        lay = bwd_layout(M, N, K, nr, dx_cut, dw_cut);
    }
    if (ws_bytes < lay.total + 256) {
        if (dw_cut.part_bytes) dw_cut = dw_plan_whole(N, K, 1);
        lay = bwd_layout(M, N, K, nr, dx_cut, dw_cut);
    }
    if (!ws || ws_bytes < lay.total + 256 || !aligned16(ws)) return MQ_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    uint8_t *base = static_cast<uint8_t *>(ws);
    const bool ep = flags & MQ_FLAG_EXTRA_PRECISION;

    // one pass over the gradients: scaled operands + c for dX, transposed sum for dW
    PrepArgs p;
    for (int i = 0; i < 3; ++i) {
        const int j = i < nr ? i : 0;
        p.dY[i] = gated ? nullptr : dY[j];
        p.GU[i] = gated ? GU[j] : nullptr;
        p.dA[i] = gated ? dA[j] : nullptr;
        p.As[i] = dX ? reinterpret_cast<uint16_t *>(base + lay.as[j]) : nullptr;
        p.lam[i] = lambda ? lambda[j] : 1.0f;
        p.mult[i] = rs[j] == 8 ? 1.0f : (float)(1 << (8 - rs[j]));
        p.bias[i] = rs[j] == 8 ? 0.0f : 128.0f;
    }
    p.alpha = alpha;
    p.zero = zero;
    p.cpart = dX ? reinterpret_cast<float *>(base + lay.cvec) : nullptr;
    // (the operand of dW is a single gradient as it stands where it is not scaled)
    const bool single = !gated && nr == 1 && p.lam[0] == 1.0f;
    const bool turn = dW && dw_turns_in_place(M, N, K, X, single ? dY[0] : nullptr, dX, dW, dX || !single, dw_cut.hb), plain_g = single && turn;
    p.G = dW && !plain_g ? reinterpret_cast<uint16_t *>(base + lay.g) : nullptr;
    p.nr = nr;
    p.M = (int)M;
    p.N = (int)N;
    p.silu = (flags & MQ_FLAG_FFN_SILU) ? 1 : 0;
    p.K = (int)K;
    p.Q = Q;
    p.QT = dX ? base + lay.qt : nullptr;
    p.turn = p.G && !turn;
    p.X = X;
    p.XT = dW && !turn ? reinterpret_cast<uint16_t *>(base + lay.xt) : nullptr;
    p.each = 0;
    p.g_step = 0;
    if (dX || p.G) {
        s = launch_prep(p, gated, st);
        if (s != MQ_OK) return s;
    }

    auto form_dx = [&]() -> mq_status {
        // slot order of the kernel: the r = 8 bit-width (if any) first
        DxArgs d;
        int order[3] = {0, 0, 0}, has8 = 0, pos = 0;
        for (int i = 0; i < nr; ++i)
            if (rs[i] == 8) {
                has8 = 1;
                order[pos++] = i;
            }
        for (int i = 0; i < nr; ++i)
            if (rs[i] != 8) order[pos++] = i;
        for (int i = 0; i < 3; ++i) {
            const int j = order[i < nr ? i : 0];
            d.As[i] = p.As[j];
            d.r[i] = rs[j];
        }
        d.QT = p.QT;
        d.cvec = p.cpart;
        d.nsplit = p.nsplit;
        d.dX = dX;
        d.M = (int)M;
        d.N = (int)N;
        d.K = (int)K;
        d.part = reinterpret_cast<float *>(base + lay.dxp);
        return launch_dx(d, dx_cut, nr, has8 != 0, ep, st);
    };
    auto form_dw = [&]() -> mq_status {
        DwArgs w{};
        w.G[0] = plain_g ? dY[0] : p.G;
        w.in_pieces = !plain_g;
        w.X = turn ? X : p.XT;
        w.dW = dW;
        w.part = reinterpret_cast<float *>(base + lay.dwp);
        w.M = (int)M;
        w.N = (int)N;
        w.K = (int)K;
        w.accumulate = (flags & MQ_FLAG_ACCUM_DW) ? 1 : 0;
        return launch_dw(w, dw_cut, turn, st);
    };
    // (operands that dW takes as they stand are not stored over by dX: dw_turns_in_place)
    const bool first = dW && !turn && dw_first(M, N, K);
    if (first) s = form_dw();
    if (s == MQ_OK && dX) s = form_dx();
    if (s == MQ_OK && dW && !first) s = form_dw();
    if (s != MQ_OK) return s;
    return launch_status();
}
}  // namespace mq

extern "C" mq_status mq_linear_bwd(const uint16_t *X, const uint8_t *Q, const float *alpha, const float *zero,
                                   const uint16_t *const *dY, const float *lambda, int64_t M, int64_t N,
                                   int64_t K, const int *rs, int nr, uint32_t flags, uint16_t *dX, float *dW,
                                   void *ws, size_t ws_bytes, void *hip_stream) {
    return mq::bwd_run(false, X, Q, alpha, zero, dY, nullptr, nullptr, lambda, M, N, K, rs, nr, flags, dX, dW, ws, ws_bytes,
                       hip_stream);
}

extern "C" mq_status mq_linear_bwd_gated(const uint16_t *X, const uint8_t *Q, const float *alpha, const float *zero,
                                         const uint16_t *const *GU, const uint16_t *const *dA, const float *lambda,
                                         int64_t M, int64_t F, int64_t K, const int *rs, int nr, uint32_t flags,
                                         uint16_t *dX, float *dW, void *ws, size_t ws_bytes, void *hip_stream) {
    if (F < 0 || F > (1 << 21)) return MQ_ERR_SHAPE;
    return mq::bwd_run(true, X, Q, alpha, zero, nullptr, GU, dA, lambda, M, 2 * F, K, rs, nr, flags, dX, dW, ws, ws_bytes,
                       hip_stream);
}

extern "C" const char *mq_status_string(mq_status status) {
    switch (status) {
        case MQ_OK: return "ok";
        case MQ_ERR_NULL: return "null pointer";
        case MQ_ERR_SHAPE: return "bad shape";
        case MQ_ERR_BITS: return "bad bit-width";
        case MQ_ERR_ALIGN: return "bad alignment";
        case MQ_ERR_WORKSPACE: return "workspace too small";
        case MQ_ERR_CAPACITY: return "overflow list capacity exceeded";
        case MQ_ERR_DEVICE: return "device error";
    }
    return "unknown status";
}
