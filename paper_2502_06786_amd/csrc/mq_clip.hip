// mq_linear_bwd_clip: gradients of the MatQuant objective with respect to the clip factors gamma, beta
// of the quantizer of section 3.1.2 (alpha = (gamma max - beta min) / 255, z = -beta min / alpha), under
// the straight-through estimator: the rounding to the 8-bit code and the rounding inside the slicing
// operator of section 3.2 pass the gradient unchanged, the clamp to 0..255 and the clamp of a slice to
// its top code pass it only where they do not act.  With u = w / alpha + z and What_r = alpha (S_r - z):
//     d What_r / d alpha = (S_r - z) - m_r w / alpha          d What_r / d z = -alpha (1 - m_r)
// where m_r = 1 where neither clamp acts.  Unlike dW, where every bit-width has the same derivative and the
// gradients are summed before one contraction, these coefficients differ per bit-width: each r takes its
// own dY_r^T X contraction (the matrix-core kernel of the backward over the tiles of all of them, into
// scratch matrices), followed by one row reduction against the coefficients (HBM-bound: 4 + 1 + 4 nr bytes
// per weight).  One preparation, one round-up of tiles and one pass over W and Q instead of one per bit-width:
// 486 -> 344 us of kernel time for 1999 tokens through 2304 x 9216 at r = 8/4/2.  A workspace with room for one scratch matrix
// (that of a call with one bit-width) serves the bit-widths one after the other, their sums over a channel kept in fp64.
#include <algorithm>

#include "mq_common.h"

namespace mq {

namespace {

struct ClipArgs {
    const float *W;       // [N, ldw]
    const uint8_t *Q;     // [N, K]
    const float *G;       // [nr][N, K]: lambda_r dY_r^T X
    const float *alpha, *zero;
    const float *gamma, *beta;  // [N] or null (= 1)
    float *dgamma, *dbeta, *dalpha, *dzero;
    double *acc;          // [N][2]: d alpha, d z of the launches before this one
    int first, last;      // of the launches of a call
    int64_t ldw;
    int N, K;
    int r[3], ep;
};

// One workgroup per output channel.  Four weights per thread and step; fp32 products, per-thread fp32
// sums over at most K / 1024 steps, fp64 across the workgroup.
template <int NR>
__global__ __launch_bounds__(256) void clip_reduce_kernel(ClipArgs a) {
    __shared__ double red[4][4];
    const int n = blockIdx.x;
    const float al = a.alpha[n], ze = a.zero[n];
    const float *w = a.W + (size_t)n * a.ldw;
    const float *g = a.G + (size_t)n * a.K;
    const uint8_t *q = a.Q + (size_t)n * a.K;
    float sa[NR], sz[NR], mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < NR; ++i) sa[i] = sz[i] = 0.f;
    for (int k = threadIdx.x * 4; k < a.K; k += 1024) {
        const f32x4 wv = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(w + k));
        f32x4 gv[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) gv[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(g + (size_t)i * a.N * a.K + k));
        const uint32_t qv = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(q + k));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // the quantizer's own operations, in its order, decide whether its clamp acted
            const float t = __fdiv_rn(wv[j], al);
            const float rounded = rintf(__fadd_rn(t, ze));
            const bool inside = rounded >= 0.0f && rounded <= 255.0f;
            const int code8 = (int)((qv >> (8 * j)) & 0xFFu);
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const int s = 8 - a.r[i], half = (1 << s) >> 1, top = (1 << a.r[i]) - 1;
                const int raw = (code8 + half) >> s;
                const bool clamped = !a.ep && raw > top;
                const float S = (float)((clamped ? top : raw) << s);
                const bool m = inside && !clamped;
                sa[i] += gv[i][j] * ((S - ze) - (m ? t : 0.0f));
                sz[i] += m ? 0.0f : gv[i][j] * -al;
            }
            mn = fminf(mn, wv[j]);
            mx = fmaxf(mx, wv[j]);
        }
    }
    double da = 0.0, dz = 0.0;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        da += sa[i];
        dz += sz[i];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        da += __shfl_xor(da, o);
        dz += __shfl_xor(dz, o);
        mn = fminf(mn, __shfl_xor(mn, o));
        mx = fmaxf(mx, __shfl_xor(mx, o));
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[wave][0] = da;
        red[wave][1] = dz;
        red[wave][2] = mn;
        red[wave][3] = mx;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    da = red[0][0] + red[1][0] + red[2][0] + red[3][0];
    dz = red[0][1] + red[1][1] + red[2][1] + red[3][1];
    if (!a.first) {
        da += a.acc[2 * n];
        dz += a.acc[2 * n + 1];
    }
    if (!a.last) {
        a.acc[2 * n] = da;
        a.acc[2 * n + 1] = dz;
        return;
    }
    const double lo = fmin(fmin(red[0][2], red[1][2]), fmin(red[2][2], red[3][2]));
    const double hi = fmax(fmax(red[0][3], red[1][3]), fmax(red[2][3], red[3][3]));
    // chain rule through alpha(gamma, beta) and z(beta, alpha), with beta min = -z alpha.  A row whose
    // clipped range is empty (the quantizer's own fp32 test) was given alpha = 1 and carries no gradient.
    const float lo32 = (float)lo, hi32 = (float)hi;
    const bool degenerate = (a.gamma ? __fmul_rn(a.gamma[n], hi32) : hi32) == (a.beta ? __fmul_rn(a.beta[n], lo32) : lo32);
    const double A = al, Z = ze;
    const double da_dg = hi / 255.0, da_db = -lo / 255.0;
    const double bmin_a2 = -Z / A;  // beta min / alpha^2
    const double dz_dg = bmin_a2 * da_dg;
    const double dz_db = -lo / A + bmin_a2 * da_db;
    if (a.dalpha) a.dalpha[n] = (float)da;
    if (a.dzero) a.dzero[n] = (float)dz;
    a.dgamma[n] = degenerate ? 0.0f : (float)(da * da_dg + dz * dz_dg);
    a.dbeta[n] = degenerate ? 0.0f : (float)(da * da_db + dz * dz_db);
}

__global__ void clip_zero_kernel(float *a, float *b, float *c, float *d, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    a[i] = 0.f;
    b[i] = 0.f;
    if (c) c[i] = 0.f;
    if (d) d[i] = 0.f;
}


}  // namespace

// the scratch matrices and what dw_each needs; never less than the backward's own workspace beside them
size_t clip_workspace_bytes(int64_t M, int64_t N, int64_t K, int nr) {
    return align256((size_t)N * K * 4 * nr) + std::max(dw_each_bytes(M, N, K, nr), mq_workspace_bytes(MQ_OP_LINEAR_BWD, M, N, K, 1)) + 512;
}

}  // namespace mq

extern "C" mq_status mq_linear_bwd_clip(const float *W, int64_t ldw, const uint16_t *X, const uint8_t *Q,
                                        const float *alpha, const float *zero, const float *gamma,
                                        const float *beta, const uint16_t *const *dY, const float *lambda, int64_t M,
                                        int64_t N, int64_t K, const int *rs, int nr, uint32_t flags, float *dgamma,
                                        float *dbeta, float *dalpha, float *dzero, void *ws, size_t ws_bytes,
                                        void *hip_stream) {
    using namespace mq;
    if (nr < 1 || nr > 3 || !rs) return MQ_ERR_BITS;
    for (int i = 0; i < nr; ++i) {
        if (rs[i] < 1 || rs[i] > 8) return MQ_ERR_BITS;
        for (int j = 0; j < i; ++j)
            if (rs[j] == rs[i]) return MQ_ERR_BITS;
    }
    if (M < 0 || N < 0 || K < 1 || ldw < K) return MQ_ERR_SHAPE;
    if (M > (1 << 22) || N > (1 << 22) || K > (1 << 22)) return MQ_ERR_SHAPE;
    if (K % 16 != 0 || N % 16 != 0 || ldw % 4 != 0) return MQ_ERR_ALIGN;
    if (N == 0) return MQ_OK;
    if (!W || !Q || !alpha || !zero || !dgamma || !dbeta || (M > 0 && (!X || !dY))) return MQ_ERR_NULL;
    for (int i = 0; i < nr && M > 0; ++i)
        if (!dY[i]) return MQ_ERR_NULL;
    if (!aligned16(W) || !aligned16(Q)) return MQ_ERR_ALIGN;
    // (a workspace that was made for more tokens may be too small for the partial tiles of fewer: dw_each then cuts nothing)
    int at_once = nr;
    size_t g_bytes = align256((size_t)N * K * 4 * nr), acc_bytes = 0;
    if (nr > 1 && ws_bytes < g_bytes + dw_each_bytes(M, N, K, nr, true) + 512) {
        at_once = 1;
        g_bytes = align256((size_t)N * K * 4);
        acc_bytes = align256((size_t)N * 2 * sizeof(double));  // (inside the room of one bit-width's backward, which holds N K codes)
    }
    const size_t used = g_bytes + acc_bytes;
    if (!ws || ws_bytes < used + dw_each_bytes(M, N, K, at_once, true) + 512 || !aligned16(ws)) return MQ_ERR_WORKSPACE;
    if (M > 0) {
        if (!aligned16(X)) return MQ_ERR_ALIGN;
        for (int i = 0; i < nr; ++i)
            if (!aligned16(dY[i])) return MQ_ERR_ALIGN;
    }
    hipStream_t st = static_cast<hipStream_t>(hip_stream);

    uint8_t *base = reinterpret_cast<uint8_t *>((reinterpret_cast<uintptr_t>(ws) + 255) & ~(uintptr_t)255);
    float *G = reinterpret_cast<float *>(base);
    if (M == 0) {  // no tokens: the objective does not depend on the weights
        clip_zero_kernel<<<dim3((unsigned)cdiv(N, 256)), dim3(256), 0, st>>>(dgamma, dbeta, dalpha, dzero, (int)N);
        return launch_status();
    }
    ClipArgs a{};
    a.W = W;
    a.Q = Q;
    a.G = G;
    a.alpha = alpha;
    a.zero = zero;
    a.gamma = gamma;
    a.beta = beta;
    a.dgamma = dgamma;
    a.dbeta = dbeta;
    a.dalpha = dalpha;
    a.dzero = dzero;
    a.ldw = ldw;
    a.N = (int)N;
    a.K = (int)K;
    a.acc = reinterpret_cast<double *>(base + g_bytes);
    a.ep = (flags & MQ_FLAG_EXTRA_PRECISION) ? 1 : 0;
    for (int i0 = 0; i0 < nr; i0 += at_once) {
        // G_r = lambda_r dY_r^T X for the bit-widths at hand, through the dW path of the backward
        mq_status s = dw_each(X, dY + i0, lambda ? lambda + i0 : nullptr, M, N, K, at_once, G, base + used, ws_bytes - used - 256, st);
        if (s != MQ_OK) return s;
        for (int i = 0; i < at_once; ++i) a.r[i] = rs[i0 + i];
        a.first = i0 == 0;
        a.last = i0 + at_once == nr;
        if (at_once == 1)
            clip_reduce_kernel<1><<<dim3((unsigned)N), dim3(256), 0, st>>>(a);
        else if (at_once == 2)
            clip_reduce_kernel<2><<<dim3((unsigned)N), dim3(256), 0, st>>>(a);
        else
            clip_reduce_kernel<3><<<dim3((unsigned)N), dim3(256), 0, st>>>(a);
        if ((s = launch_status()) != MQ_OK) return s;
    }
    return MQ_OK;
}
