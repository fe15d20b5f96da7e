// Internal interface of the linear-layer kernels (not part of the public ABI): tile loads, code conversions, and the
// main loop that the forward kernels share.
#pragma once

#include <type_traits>
#include <utility>

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

// f(integral_constant 0), ..., f(integral_constant N - 1): the schedules below are written out at compile time
template <int... I, typename F>
__device__ __forceinline__ void static_for_each(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_each(std::make_integer_sequence<int, N>{}, f);
}

// acc += A B on the 16x16x32 product, in place in the accumulator file.  The large kernels are bound by the power that the chip
// draws, and of the two bf16 shapes this one does more work for it: a loop of products alone, operands from LDS, one wave per
// SIMD, runs at 1.93 PFLOP/s on N(0, 1) values (32x32x16: 1.71), at 2.28 with small codes as A (1.76; codes as B: 2.07), which is
// why codes are A everywhere.  14336 x 3584, 8192 tokens, r = 8/4/2: forward with the objective 2050 -> 1900 us, dX 2000 -> 1790,
// dW 685 -> 625 (the clock rises from 1.72 to 2.0 GHz).  In assembly because the register allocator, given the
// builtin, does not keep 240 and more accumulator registers in place: it moved them about with hundreds of copies per stage.
// The compiler does not see a matrix product here, so the waits it would place are ours: an operand written by a vector
// instruction (not one read from LDS) is used two wait states later at the earliest, and an accumulator is read or copied eight
// wait states after its product at the earliest.  The schedules keep the last two products of a step free of conversions (not those
// whose last conversions belong to a bit-width that the next step comes to five products later), and
// mfma16_settle() stands behind the last product of a stage (the matrix core is still busy then).  Copies that the register
// allocator makes are its own choice: tests/test_matrix_waits.py follows every path through the compiled kernels, over the ends
// of loops too, and fails where one comes too close.  (Two wait states inside the assembly of the first product of each step
// would rule out most of that and cost 0.1 of 14.0 us with 77 tokens on 4096 x 4096, 0.5 of 187 us on the largest single forward.)
// FILE_A: the accumulator file or (where two workgroups share a compute unit and it holds 128 registers) the vector file.
template <bool FILE_A = true>
__device__ __forceinline__ void mfma16_acc(f32x4 &acc, const u32x4 &a, const u32x4 &b) {
    if constexpr (FILE_A)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma16_settle() {
    asm volatile("s_nop 7");
    __builtin_amdgcn_sched_barrier(0);
}

// ---- LDS tiles ------------------------------------------------------------------------------
// bf16 tile: ROWS x 64 elements, 128-byte rows of eight 16-byte chunks; chunk c of row r is stored
// at chunk position c ^ ((r >> 1) & 7).  u8 tile: ROWS x 64 bytes, four chunks per row; chunk c of
// row r at position c ^ ((r >> 2) & 3).  The LDS has 64 four-byte banks and serves a 16-byte read
// sixteen lanes at a time, so sixteen consecutive rows must land on sixteen distinct 16-byte bank
// groups of a 256-byte window; both swizzles do that (measured: same rate as a contiguous read).  A direct-to-LDS load writes lane l of a wave at base + 16 l, so the swizzle is
// applied by choosing which global chunk each lane fetches.

// The operands of the 16x16x32 product are read with sixteen rows across the lanes and four chunks of them across the groups of
// sixteen lanes, and those served together are lanes 0-3, 12-15, 20-23, 24-27 (4-11, 16-19, 28-31; the upper half likewise): rows
// 0-3 and 12-15 of one group, 4-11 of its neighbour.  The chunks of neighbouring groups therefore have to differ in the right
// bits: with chunk g for group g every read met a conflict (half of the cycles the LDS was busy).  Which elements of the
// contraction a group takes is free as long as both operands agree.
__device__ __forceinline__ int group_chunk(int g4) { return (0x9C >> (2 * g4)) & 3; }  // 0, 3, 1, 2

// 16 bytes per lane, from `offset` (per lane) behind a descriptor's base, to `at` + 16 lane in LDS.  In assembly because
// the compiler lets a transposing read wait for all direct-to-LDS loads that it has seen, those of the stages that are to
// stay on their way too (stage_barrier waits for the right ones).  It writes no register but m0, which nothing else uses in a kernel
// that loads its tiles with it alone (the compiler refuses it in the list of clobbered registers).  One wait state covers m0.  A
// descriptor is fixed by scalar_rsrc(), in case the compiler gets it there with vector instructions (kDescriptorWait wait states to a
// load that reads it): they stand in load_to_lds; a schedule that uses the pieces counts the instructions between descriptor and load.
constexpr int kDescriptorWait = 5;
__device__ __forceinline__ u32x4 scalar_rsrc(const void *base, int bytes) {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    u32x4 rsrc = {(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)p), (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(p >> 32)) & 0xFFFFu,
                  (uint32_t)__builtin_amdgcn_readfirstlane(bytes), 0x00020000u};
    asm volatile("" : "+s"(rsrc));
    return rsrc;
}
__device__ __forceinline__ void load_to_lds(const u32x4 &rsrc, uint32_t offset, uint32_t at) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(offset), "s"(rsrc), "s"(at) : "memory");
}
// the same in two pieces for a schedule that puts a matrix product (and so a wait state) between them
template <int PLUS>
__device__ __forceinline__ void aim_load_to_lds(uint32_t at) {
    asm volatile("s_add_u32 m0, %0, %1" ::"s"(at), "n"(PLUS) : "scc");
}
__device__ __forceinline__ void aimed_load_to_lds(const u32x4 &rsrc, uint32_t offset) {
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(offset), "s"(rsrc) : "memory");
}

// Four elements of one column per lane from a tile whose rows are the contraction index: a transposing read takes 8 bytes from every lane,
// so sixteen lanes bring four rows of sixteen elements (four lanes a row), and gives each of them one column of those rows.
__device__ __forceinline__ u32x2 read_turned16(const uint8_t *at) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 *lds_s16x4;
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(at)));
}

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
// r-bit slice of section 3.2 as bf16(128 + code), two codes at a time.
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

// Four codes (one dword) -> two dwords of bf16 pairs, in four steps of two independent instructions each, so that a step fits
// behind a matrix product without waiting for the one before it (a wave issues a dependent vector instruction only every eight
// cycles, and a 16x16x32 product takes sixteen).  t carries the values between the steps; the empty asm keeps a step where it is.
// A code of r = 2 depends on the upper three bits of the byte alone, rounding and clamp included: KIND_2 looks four of them up with one
// byte permutation, five instructions instead of eight.  The operand's bits are the same.  Whole calls with the look-up against calls without
// at 2670 pairs of times (512 to 14336 rows and columns, 17 to 4096 tokens): r = 2 alone dX 0.965 times as long, forward 0.971 (with the
// objective 0.975); r = 8/2 dX 0.975, forward in whole tiles 0.973 (0.984); 4/2 dX 0.986, forward 0.990 (0.993); 8/4/2 forward 0.992
// (0.989; tiles of 64 and 96 tokens 0.994 (0.988), 1.7 % longer at worst), dX 0.992 to 0.996 up to 96 tokens a tile and level above
// (launch_dx_mb).
enum CodeKind { KIND_ANY, KIND_8, KIND_2 };
constexpr CodeKind code_kind(bool is8, bool is2) { return is8 ? KIND_8 : is2 ? KIND_2 : KIND_ANY; }
template <CodeKind KIND, bool EP, int STEP>
__device__ __forceinline__ void convert_step(uint32_t d, const SliceParam &p, uint32_t (&t)[4], uint32_t &lo, uint32_t &hi) {
    if constexpr (KIND == KIND_2) {
        if constexpr (STEP == 0) t[0] = d >> 5;
        if constexpr (STEP == 1) t[0] &= 0x07070707u;
        if constexpr (STEP == 2) t[0] = __builtin_amdgcn_perm(EP ? 0x04030302u : 0x03030302u, 0x02010100u, t[0]);
        if constexpr (STEP == 3) {
            lo = __builtin_amdgcn_perm(kMagic128, t[0], 0x05010500u);   // (byte 5 of the pair: 0x43)
            hi = __builtin_amdgcn_perm(kMagic128, t[0], 0x05030502u);
            asm volatile("" : "+v"(lo), "+v"(hi));
        } else {
            asm volatile("" : "+v"(t[0]));
        }
    } else if constexpr (KIND == KIND_8) {  // int8 -> fp32 -> bf16 (exact, codes <= 255)
        if constexpr (STEP < 2) {
            t[2 * STEP] = __float_as_uint((float)((d >> (16 * STEP)) & 0xFFu));
            t[2 * STEP + 1] = __float_as_uint((float)((d >> (16 * STEP + 8)) & 0xFFu));
            asm volatile("" : "+v"(t[2 * STEP]), "+v"(t[2 * STEP + 1]));
        } else if constexpr (STEP == 2) {
            lo = __builtin_amdgcn_perm(t[1], t[0], 0x07060302u);
            hi = __builtin_amdgcn_perm(t[3], t[2], 0x07060302u);
            asm volatile("" : "+v"(lo), "+v"(hi));
        }
    } else {
        if constexpr (STEP == 0) {
            t[0] = __builtin_amdgcn_perm(0u, d, EP ? 0x0C010C00u : 0x010C000Cu);
            t[1] = __builtin_amdgcn_perm(0u, d, EP ? 0x0C030C02u : 0x030C020Cu);
        } else if constexpr (STEP == 1) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
                t[c] = EP ? t[c] + p.half2
                          : __builtin_bit_cast(uint32_t, __builtin_elementwise_add_sat(__builtin_bit_cast(u16x2, t[c]),
                                                                                       __builtin_bit_cast(u16x2, p.half2)));
        } else if constexpr (STEP == 2) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const unsigned short s16 = (unsigned short)p.sh;
                t[c] = EP ? t[c] >> p.sh : __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, t[c]) >> u16x2{s16, s16});
            }
        } else {
            lo = (EP ? t[0] & 0x00FF00FFu : t[0]) | kMagic128;
            hi = (EP ? t[1] & 0x00FF00FFu : t[1]) | kMagic128;
            asm volatile("" : "+v"(lo), "+v"(hi));
        }

    }
}
// What stands between the products of one 32-wide step, laid out at compile time.  A product takes the matrix core sixteen cycles
// and a wave issues an instruction every four, so up to three instructions fit behind each without cost, and a fourth one that
// another product could have had idles the matrix core.
//   NM products, GROUP of them per block of 16 tokens (BLOCKS blocks); PAIRS dwords of codes to convert for the next step, those
//   at multiples of PERIOD by the route of r = 8 if HAS8 (three conversion steps instead of four); STEP 0 or 1 of the stage;
//   LOADS global loads and CODES reads of the next stage's code bytes: in LONG stages the former over both steps and the latter
//   early in step 0; in short ones, in which loads are waited for, the former in step 0, and the latter once the bytes of this stage
//   are used up, which saves copying them;
//   IN_PLACE: the operands of a token block are read at its last product, otherwise at the first BLOCKS products;
//   LOW: tiles of up to 64 tokens, where a stage is as long as its instructions and its loads take and the products wait for
//   both: the loads go behind the first products, before the conversions there;
//   FREE: products at the end of a step without conversions behind them (mfma16_acc).
template <int NM, int GROUP, int BLOCKS, int PAIRS, int PERIOD, bool HAS8, int STEP, int LOADS, bool LONG, int CODES, bool IN_PLACE,
          bool LOW, int FREE>
struct StepSchedule {
    int conv[NM + 1] = {};                // conversion steps before product q
    int load[NM + 1] = {}, code[NM + 1] = {};
    int pair[4 * PAIRS] = {}, step[4 * PAIRS] = {}, at[4 * PAIRS] = {};   // the conversion steps in their order
    int width = 1;                        // pairs converted side by side
    int first_load = 0;                   // loads of the steps before

    constexpr StepSchedule() {
        int uses[NM] = {};
        for (int q = 0; q < NM; ++q) {
            load[q + 1] = load[q];
            code[q + 1] = code[q];
            for (int l = 0; l < LOADS; ++l) {
                const int block = l * (LONG ? 2 : 1) * BLOCKS / LOADS;
                const int behind = !LOW ? block % BLOCKS * GROUP + 1 : NM < 2 * LOADS ? 0 : l;
                if (block / BLOCKS == STEP && behind == q) ++load[q + 1], uses[q] += 3;
                if (q == 0 && block / BLOCKS < STEP) ++first_load;
            }
            for (int e = 0; STEP == 0 && e < CODES; ++e)
                if ((LONG ? e * GROUP + GROUP / 2 : NM - 2 - CODES + e) == q) ++code[q + 1], ++uses[q];
            if (IN_PLACE ? q % GROUP == GROUP - 1 : q < BLOCKS) uses[q] += 2;
        }
        int total = 0;
        for (int e = 0; e < PAIRS; ++e) total += HAS8 && e % PERIOD == 0 ? 3 : 4;
        // room for conversion steps behind each product, at the least number of instructions per product for which they all fit;
        // they are dealt out in proportion to it.
        int room[NM] = {}, rooms = 0, seen = 0, most = 1;
        for (int budget = 3; rooms < total; ++budget) {
            rooms = 0;
            for (int q = 0; q < NM; ++q) rooms += room[q] = q < NM - FREE && uses[q] < budget ? (budget - uses[q]) / 2 : 0;
        }
        for (int q = 0; q < NM; ++q) {
            seen += room[q];
            conv[q + 1] = total * seen / rooms;
            if (conv[q + 1] - conv[q] > most) most = conv[q + 1] - conv[q];
        }
        while (width < PAIRS && (width < most || PAIRS % width != 0)) ++width;
        int n = 0;
        for (int g = 0; g < PAIRS; g += width)
            for (int s = 0; s < 4; ++s)
                for (int w = 0; w < width; ++w)
                    if (s < 3 || !(HAS8 && (g + w) % PERIOD == 0)) pair[n] = g + w, step[n] = s, at[n++] = w;
    }
};
// all four steps at once (prologues)
template <CodeKind KIND, bool EP>
__device__ __forceinline__ u32x4 convert_eight(uint32_t d0, uint32_t d1, const SliceParam &p) {
    uint32_t o[4], t[4];
    static_for<8>([&](auto c_tag) {
        constexpr int c = decltype(c_tag)::value, half = c / 4;
        convert_step<KIND, EP, c % 4>(half ? d1 : d0, p, t, o[2 * half], o[2 * half + 1]);
    });
    return u32x4{o[0], o[1], o[2], o[3]};
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
    uint32_t *arrived;  // workgroups that have left their sums (the launch before has cleared it); the last one finishes the losses.
                        // Null: a launch of its own does
    float *losses;      // in the caller's order, in which bit-width i has slot loss_slot[i]
    int loss_slot[3];
    float inv_mn;
    const float *bias;  // [N] added to every output before it is rounded, or null
    // plain kernels only: the layer is the stacked gate / up projection of a gated unit (channels (g, u) pairs)
    // and A[i] [M, N / 2] receives act(g) u of the rounded outputs; gate = 0 none, 1 GELU-tanh, 2 SiLU
    uint16_t *A[3];
    int gate;
};

// Where an accumulator lives: with three bit-widths and 96 tokens two workgroups share a compute unit, each with 128 accumulator
// registers, and four of the 36 blocks go to the vector file; so do the few of one bit-width in low tiles, where the vector file has
// room and copies between two pieces of code are not needed.
constexpr bool fwd_acc_in_file_a(int nr, int mb, int i, int tb) { return !(nr == 3 && mb == 3 && tb == 5 && i > 0) && !(nr == 1 && mb <= 2); }

// The contraction of one workgroup: acc[i][rb][tb] = sum over k in [64 kt0, k_end) of code_i[channels 16 rb .. of this wave][k] *
// X[tokens m0 + 16 tb ..][k], for all bit-widths i and token blocks tb of the tile at (m0, n0) (LAST2: the last
// bit-width is 2).  Four waves; wave w owns
// channels [32 w, 32 w + 32) of the tile for all its tokens; lane (l16, g4) ends up with channels 4 g4 .. 4 g4 + 3 of token l16 of
// a block.  ROWSUM: also rsum[j] += this thread's share (chunk t % 8 of
// row t / 8) of sum_k X for the token blocks in rs_mask.
template <int NR, bool HAS8, bool LAST2, bool EP, int MB, bool ROWSUM, typename Args>
__device__ __forceinline__ void fwd_main_loop(const Args &a, uint8_t *smem, int m0, int n0, int kt0, int nkt, int k_end,
                                              f32x4 (&acc)[NR][2][2 * MB], float (&rsum)[MB], uint32_t rs_mask) {
    constexpr int BM = 32 * MB;
    constexpr int X_TILE = BM * 128;
    constexpr int STAGE = X_TILE + FWD_Q_TILE;
    constexpr int LPS = MB + 2;  // direct-to-LDS loads per wave and stage
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g4 = lane >> 4, l16 = lane & 15;

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

    // LDS fragment addresses (byte offsets inside a stage).  The order of the contraction inside a stage is free as long as both
    // operands follow it: a lane reads the sixteen code bytes 16 gc .. of a row at once and uses eight of them per 32-wide step.
    const int nl = wave * 32 + l16;
    const int gc = group_chunk(g4);
    const uint32_t qa = X_TILE + nl * 64 + ((gc ^ ((nl >> 2) & 3)) << 4);   // + 1024 per block of 16 channels
    uint32_t xa[2];                                                         // + 2048 per block of 16 tokens
#pragma unroll
    for (int t = 0; t < 2; ++t) xa[t] = l16 * 128 + (((2 * gc + t) ^ ((l16 >> 1) & 7)) << 4);

    SliceParam sp[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) sp[i] = slice_param<EP>(a.r[i]);

#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int tb = 0; tb < 2 * MB; ++tb) acc[i][rb][tb] = f32x4{0.f, 0.f, 0.f, 0.f};

    issue(0);
    issue(1);
    issue(2);
    // stage 0 must have landed before the first operand fetch; stages 1 and 2 may stay in flight
    stage_barrier<2 * LPS, 0>();

    // Activation operands.  A block of tokens is done with after 2 NR products, and where the next block of the same step keeps
    // the matrix core busy for long enough its register is refilled for the next step right there; the smallest tiles have a
    // second set, which is requested from the first product on.
    constexpr int XS = (NR == 1 || MB <= 2) ? 2 : 1;
    u32x4 xf[XS][2 * MB];
    u32x4 raw[2];          // the sixteen code bytes of this lane's two channels: both steps of one stage
    u32x4 wf[2][NR][2];    // code operands of the two steps of a stage
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) raw[rb] = *reinterpret_cast<const u32x4 *>(smem + qa + rb * 1024);
#pragma unroll
    for (int tb = 0; tb < 2 * MB; ++tb) xf[0][tb] = *reinterpret_cast<const u32x4 *>(smem + xa[0] + tb * 2048);
    static_for<NR>([&](auto i_tag) {
        constexpr int i = decltype(i_tag)::value;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
            wf[0][i][rb] = convert_eight<code_kind(HAS8 && i == 0, LAST2 && i == NR - 1), EP>(raw[rb][0], raw[rb][1], sp[i]);
    });

    // One stage of 64 k: two 32-wide steps of 4 NR MB MFMAs.  A wave issues in order, so whatever
    // is queued behind an MFMA that waits for the matrix pipe waits with it; the other work of a
    // step is therefore cut into small pieces (StepSchedule), fenced so that the compiler keeps them between the MFMAs: the
    // conversions of the next step's code operands, the reads of its activation operands, the global loads of stage kt + 3, in
    // step 0 the code bytes of the next stage.  (After the last stage that is a stage of zeros,
    // which nobody multiplies: a copy of the code for the last stage makes the compiler move accumulators between the two.  One
    // bit-width in low tiles has that copy, MORE = false: its accumulators are few, and a range of K is five to ten stages, of
    // which the one that prepares nothing is 0.1 us shorter.)
    // (LOW at two bit-widths: 4096 x 4096, 19 tokens 14.6 -> 14.9 us, 1712 x 1184 8.9 -> 9.0)
    constexpr bool LOW = MB <= 2 && NR != 2, APART = LOW && NR == 1;
    auto tile = [&](int kt, auto more_tag) {
        constexpr bool MORE = decltype(more_tag)::value;
        constexpr int NM = 4 * NR * MB;
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
        static_for<2>([&](auto t_tag) {
            constexpr int t = decltype(t_tag)::value;
            constexpr StepSchedule<NM, 2 * NR, 2 * MB, 4 * NR, NR, HAS8, t, LPS, NR * MB >= 12, 2, XS == 1, LOW, LOW && NR == 3 ? 0 : 2> plan;
            constexpr bool PREPARE = MORE || t == 0;   // there is a next step
            const uint8_t *src = t == 0 ? cur + xa[1] : nxt + xa[0];
            uint32_t tmp[plan.width][4];
            auto loads = [&](auto q_tag) {
                constexpr int q = decltype(q_tag)::value;
                static_for<MORE ? plan.load[q + 1] - plan.load[q] : 0>([&](auto u_tag) {
                    issue_one(kt + 3, plan.first_load + plan.load[q] + decltype(u_tag)::value);
                });
            };
            static_for<NM>([&](auto q_tag) {
                constexpr int q = decltype(q_tag)::value, tb = q / (2 * NR), i = q % (2 * NR) / 2, rb = q % 2;
                mfma16_acc<fwd_acc_in_file_a(NR, MB, i, tb)>(acc[i][rb][tb], wf[t][i][rb], xf[t % XS][tb]);
                if constexpr (PREPARE && XS == 2 && q < 2 * MB) xf[1 - t % XS][q] = *reinterpret_cast<const u32x4 *>(src + q * 2048);
                if constexpr (PREPARE && XS == 1 && q % (2 * NR) == 2 * NR - 1) xf[0][tb] = *reinterpret_cast<const u32x4 *>(src + tb * 2048);
                if constexpr (LOW) loads(q_tag);
                static_for<MORE ? plan.code[q + 1] - plan.code[q] : 0>([&](auto u_tag) {
                    constexpr int e = plan.code[q] + decltype(u_tag)::value;
                    rawn[e] = *reinterpret_cast<const u32x4 *>(nxt + qa + e * 1024);
                });
                static_for<PREPARE ? plan.conv[q + 1] - plan.conv[q] : 0>([&](auto u_tag) {
                    constexpr int c = plan.conv[q] + decltype(u_tag)::value, pair = plan.pair[c], step = plan.step[c];
                    constexpr int ci = pair % NR, crb = pair / NR / 2, half = pair / NR % 2;
                    u32x4 &out = wf[1 - t][ci][crb];
                    uint32_t lo = out[2 * half], hi = out[2 * half + 1];
                    convert_step<code_kind(HAS8 && ci == 0, LAST2 && ci == NR - 1), EP, step>(t == 0 ? raw[crb][2 + half] : rawn[crb][half], sp[ci], tmp[plan.at[c]], lo, hi);
                    if constexpr (step == (HAS8 && ci == 0 ? 2 : 3)) {
                        out[2 * half] = lo;
                        out[2 * half + 1] = hi;
                    }
                });
                if constexpr (!LOW) loads(q_tag);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        mfma16_settle();
        if constexpr (MORE) {
            raw[0] = rawn[0];
            raw[1] = rawn[1];
        }
    };

    for (int kt = 0; kt < nkt - (APART ? 1 : 0); ++kt) {
        // Stage kt + 1 must be resident for the operand prefetch of this iteration; the
        // loads of stage kt + 2 may stay in flight.  After the barrier every wave is done with
        // stage kt - 1, whose buffer stage kt + 3 reuses.
        stage_barrier<LPS, 2 * MB>();
        tile(kt, std::true_type{});
    }
    if constexpr (APART) tile(nkt - 1, std::false_type{});  // (resident since the barrier of the stage before, or of the prologue)
    wait_vm0();  // zero-fill loads of dead stages must not land in the staging area below
}

// Ends a workgroup of a kernel that evaluates the objective: its sums (`v` of slot t in thread t < 4) go to a.partial.  With a counter
// (kLossArrivals), the workgroup that finds all others arrived adds them, in the order of the workgroups whichever it is, and writes the
// losses.  Nobody waits for anybody.  The sums and the counter are written and read past the caches that XCDs do not share (agent scope);
// the sums are there before the counter counts them because the wave waits for its stores in between.  (workgroups: of the launch.  Asked of
// gridDim it would add 256 bytes to the arguments of every launch of a kernel that asks for nothing else there.)
template <int NR, typename Args>
__device__ __forceinline__ void leave_sums(const Args &a, float v, uint32_t workgroups, float *partial, uint32_t *arrived) {
    static_assert(kLossArrivals <= 64, "one wave adds the sums, a workgroup's in a lane");
    if (threadIdx.x >= 64) return;
    if (!arrived) {
        if (threadIdx.x < 4) partial[(size_t)blockIdx.x * 4 + threadIdx.x] = v;
        return;
    }
    if (threadIdx.x < 4) __hip_atomic_store(partial + (size_t)blockIdx.x * 4 + threadIdx.x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_vm0();
    uint32_t before = 0;
    if (threadIdx.x == 0) before = __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(before) != workgroups - 1) return;
    wait_vm0();   // (nothing below is loaded before the count is known)
    double sum[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i)
        sum[i] = threadIdx.x < workgroups ? (double)__hip_atomic_load(partial + (size_t)threadIdx.x * 4 + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum[i] += __shfl_xor(sum[i], o, 64);
    if ((int)threadIdx.x < NR) {
        const int slot = threadIdx.x == 0 ? a.loss_slot[0] : threadIdx.x == 1 ? a.loss_slot[1] : a.loss_slot[2];
        double mine = sum[0];
#pragma unroll
        for (int i = 1; i < NR; ++i) mine = slot == i ? sum[i] : mine;
        a.losses[threadIdx.x] = (float)(mine * (double)a.inv_mn);
    }
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
    float *part;            // splits > 1: fp32 accumulators, [split][tile][block of 16 k][block of 16 tokens][256] quads
};

DxPlan dx_plan(int64_t M, int64_t N, int64_t K, int nr);
// the forward at one bit-width (plain or gated), mb as fwd_wide_mb has chosen it
mq_status launch_fwd_wide(const FwdArgs &f, int mb, bool has8, bool ep, hipStream_t st);
// whether the kernels have a form for bit-widths in slot order with r = 2 last: 2, any two and 8/./2
constexpr bool has_last2(int nr, bool has8) { return nr == 2 || (nr == 1) != has8; }
mq_status launch_dx(DxArgs d, const DxPlan &plan, int nr, bool has8, bool ep, hipStream_t st);

}  // namespace mq
