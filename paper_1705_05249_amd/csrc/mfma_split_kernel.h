// FP32 macro-tile GEMM kernel on the bf16 matrix pipes.
//
// Every FP32 element is the sum of three bf16 values, x = x1 + x2 + x3 (each the rounded rest of the one before: 3 x 8
// significand bits and their signs hold all 24), and of the nine products of two such elements all but a3 b3 are taken:  a1 b1 +
// (a1 b2 + a2 b1 + a2 b2 + a1 b3 + a3 b1 + a2 b3 + a3 b2).  With |x2| <= 2^-8 |x| and |x3| <= 2^-17 |x| the one left out is at most 2^-34
// of |a b|; a2 b3 + a3 b2 reach 2^-24, what rounding a b to FP32 costs (without them a sum that one product dominates was off by
// up to 0.95 units in its last place; with them 0.506, FP32 pipes 0.5).  Products of bf16 values are exact in the matrix pipes' FP32
// accumulators; a1 b1 has accumulators of its own, the seven small products share others that are added once at the end, so the large
// sums see one rounding per four values of k (v_mfma_f32_32x32x16_bf16) where v_mfma_f32_32x32x2_f32 rounds for each.  Eight bf16
// instructions of 32 cycles take the place of eight FP32 ones of 64 (16 values of k).
//
// Elements are multiplied by 2^20 on their way into the parts, so that the last bit of any FP32 value, 2^-149, lies above bf16's
// smallest one, 2^-133: no part loses bits, subnormal elements included.  (2^16 would do for that, but the pipes align products of subnormal
// factors by their exponents: elements around 2^-140 0.62 units in the last place.)  The sums are 2^40 times too large until the end.  What they
// cannot hold, elements from 2^107 and sums from 2^88 on, Inf and NaN, leaves Inf or NaN in a rest or an accumulator: a work-group that finds
// one computes its tile again with the FP32 instructions.  (While elements were taken as they are, one below 2^-110 in a tile's operands cost
// it the second computation: 4096^3 of values around 1e-36 1219 us, now 749, 2048^3 216, now 128; values near one 738 -> 752 us, 106 -> 108.)
//
// Structure: global -> registers -> (split) -> LDS, two LDS stages of 32 values of k, DEPTH K-tiles in flight in staging
// registers; one barrier per K-tile; issue order pinned slot by slot, one MFMA per slot.
#pragma once

#include "mfma_kernel.h"

namespace mg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef short shortx4 __attribute__((ext_vector_type(4)));

// two elements, scaled -> their three parts, packed
constexpr float SPLIT_SCALE = 0x1p20f, SPLIT_UNSCALE = 0x1p-40f;
struct SplitPair {
    uint32_t part[3];
};
__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{a, b}), bf16x2));
}
// (beyond: set when an element is Inf, NaN or too large for its leading part.  Two instructions of the accumulators' test would do
// instead, but without this one the compiler moves the splits out of their slots and spills 30 registers: 4096^3 800 us.)
__device__ __forceinline__ SplitPair split_pair(float a, float b, bool &beyond)
{
    SplitPair s;
    a *= SPLIT_SCALE;
    b *= SPLIT_SCALE;
    s.part[0] = bf16_pair(a, b);
    a -= __builtin_bit_cast(float, s.part[0] << 16);
    b -= __builtin_bit_cast(float, s.part[0] & 0xffff0000u);
    s.part[1] = bf16_pair(a, b);
    a -= __builtin_bit_cast(float, s.part[1] << 16);
    b -= __builtin_bit_cast(float, s.part[1] & 0xffff0000u);
    s.part[2] = bf16_pair(a, b);
    constexpr int NOT_FINITE = 0x207;
    beyond |= __builtin_amdgcn_classf(a, NOT_FINITE) | __builtin_amdgcn_classf(b, NOT_FINITE);
    return s;
}
// ---- one operand tile: ROWS rows x 32 values of k ---------------------------------------------------
// LDS: three planes (one per part).  Operand along k: [row][k], 64-byte rows of four 16-byte chunks, swizzled; along its
// rows: [k][row] as in memory, read with the transposing ds_read_b64_tr_b16 (lds_layout.h).
template <int ROWS, int NT, bool KCONTIG, bool EDGE, int DEPTH> struct SplitLoader {
    static constexpr int BK = 32;
    static constexpr int LOADS = ROWS * BK / 4 / NT;                    // 16-byte pieces per thread
    static constexpr int PLANE = ROWS * BK * 2;
    static constexpr int STAGE = 3 * PLANE;
    static constexpr int RCH = ROWS / 4;                                 // pieces per line of an operand along its rows
    static_assert(LOADS >= 1 && ROWS * BK / 4 % NT == 0, "whole pieces per thread");
    static_assert(ROWS >= 128, "the [k][row] planes' lines are whole bank rows");
    static constexpr uint32_t OUT_OF_RANGE = 0x80000000u;

    u32x4 regs[DEPTH][LOADS];
    uint32_t goff[LOADS];
    int slot[LOADS];                // LDS byte offset of each piece inside a plane
    bool keep[4];                   // EDGE, along the rows: element e of this lane's pieces is a row that exists
    bool beyond;                    // see split_pair
    SplitPair made[2];              // the piece being split

    __device__ __forceinline__ void prepare(int64_t ld, int rows, int t)
    {
        beyond = false;
        static_for<LOADS>([&](auto Qc) {
            constexpr int Q = decltype(Qc)::value;
            const int idx = t + Q * NT;
            if constexpr (KCONTIG) {
                const int r = idx / 8, c = idx % 8;
                goff[Q] = static_cast<uint32_t>((r * ld + c * 4) * 4);
                slot[Q] = ldsmap::split_row_slot(r, c / 2) + 8 * (c % 2);
            } else {
                const int mc = idx % RCH, l = idx / RCH;
                goff[Q] = !EDGE || mc * 4 < rows ? static_cast<uint32_t>((mc * 4 + l * ld) * 4) : OUT_OF_RANGE;
                slot[Q] = ldsmap::transposed_slot(ROWS, l, mc / 2) + 8 * (mc % 2);
            }
        });
        // (pieces of a thread are whole lines apart: the same rows)
        static_assert(KCONTIG || NT % RCH == 0, "pieces of a thread cover the same rows");
#pragma unroll
        for (int e = 0; e < 4; ++e) keep[e] = !EDGE || KCONTIG || (t % RCH) * 4 + e < rows;
    }

    // Descriptor of the tile of `rows` rows and `ks` (<= 32) values of k from (r0, l0) on: it ends with the last element
    // that exists, and a load past its end returns zeros without touching memory (ks <= 0: all of them).
    __device__ __forceinline__ static __amdgpu_buffer_rsrc_t aim(const float *X, int64_t ld, int64_t r0, int64_t l0, int rows, int ks)
    {
        const float *base = KCONTIG ? X + r0 * ld + l0 : X + r0 + l0 * ld;
        if (ks > BK) ks = BK;
        const int64_t extent = KCONTIG ? (rows - 1) * ld + ks : (ks - 1) * ld + rows;
        const int range = static_cast<int>(extent * 4) & -static_cast<int>(ks > 0);      // (no branch: it would cut the K loop's schedule)
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, range, 0x00020000);
    }
    template <int SET, int Q> __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rsrc)
    {
        regs[SET][Q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, goff[Q], 0, 0);
    }
    // values of k beyond the sum (operand along k: they are the next row's)
    template <int SET, int Q> __device__ __forceinline__ void cut(int ks, int t)
    {
        if constexpr (KCONTIG) {
            const int c = (t + Q * NT) % 8;
#pragma unroll
            for (int e = 0; e < 4; ++e) regs[SET][Q][e] = c * 4 + e < ks ? regs[SET][Q][e] : 0u;
        }
    }
    template <int SET, int Q, int HALF> __device__ __forceinline__ void split()
    {
        float v[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            uint32_t bits = regs[SET][Q][2 * HALF + e];
            if constexpr (EDGE && !KCONTIG) bits = keep[2 * HALF + e] ? bits : 0u;
            v[e] = __builtin_bit_cast(float, bits);
        }
        made[HALF] = split_pair(v[0], v[1], beyond);
    }
    // the staged floats themselves -> LDS, and a fragment (4 values of k per lane of K-step `step`) of them, as in mfma_kernel.h
    __device__ __forceinline__ void store_floats(char *stage, int t) const
    {
        static_for<LOADS>([&](auto Qc) {
            constexpr int Q = decltype(Qc)::value;
            const int idx = t + Q * NT;
            u32x4 v = regs[0][Q];
            if constexpr (EDGE && !KCONTIG) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = keep[e] ? v[e] : 0u;
            }
            if constexpr (KCONTIG) *reinterpret_cast<u32x4 *>(stage + ldsmap::kcontig_slot<32>(idx / 8, idx % 8)) = v;
            else *reinterpret_cast<u32x4 *>(stage + ldsmap::native_slot(ROWS, idx / RCH, idx % RCH)) = v;
        });
    }
    __device__ __forceinline__ static u32x4 read_floats(const char *stage, int lane, int wrow, int f, int step)
    {
        if constexpr (KCONTIG) {
            return *reinterpret_cast<const u32x4 *>(stage + ldsmap::kcontig_slot<32>(wrow + 32 * f + lane % 32, 2 * step + lane / 32));
        } else {
            const char *p = stage + ldsmap::native_base(ROWS, lane, wrow, f) + 8 * step * 4 * ROWS;
            return u32x4{*reinterpret_cast<const uint32_t *>(p), *reinterpret_cast<const uint32_t *>(p + 4 * ROWS),
                         *reinterpret_cast<const uint32_t *>(p + 8 * ROWS), *reinterpret_cast<const uint32_t *>(p + 12 * ROWS)};
        }
    }
    template <int Q> __device__ __forceinline__ void store(char *stage)
    {
#pragma unroll
        for (int p = 0; p < 3; ++p)
            *reinterpret_cast<u32x2 *>(stage + p * PLANE + slot[Q]) = u32x2{made[0].part[p], made[1].part[p]};
    }
};

// Fragments of one operand: F blocks of 32 rows from row `wrow` on; lane l holds row l % 32, values 8 (l / 32) .. + 7 of the 16 of K-step s
template <int ROWS, bool KCONTIG, int F> struct SplitFragments {
    static constexpr int PLANE = ROWS * 64;
    int at[KCONTIG ? 2 : F];
    __device__ __forceinline__ void prepare(int lane, int wrow, int offset)
    {
        if constexpr (KCONTIG) {
            const int r = wrow + lane % 32;
            at[0] = offset + ldsmap::split_row_slot(r, lane / 32);
            at[1] = offset + ldsmap::split_row_slot(r, 2 + lane / 32);
        } else {
#pragma unroll
            for (int f = 0; f < F; ++f) at[f] = offset + ldsmap::split_line_base(ROWS, lane, wrow + 32 * f);
        }
    }
    template <int S, int FI, int PART> __device__ __forceinline__ u32x4 read(const char *lds, int stage) const
    {
        if constexpr (KCONTIG) {
            return *reinterpret_cast<const u32x4 *>(lds + at[S] + stage + PART * PLANE + FI * 2048);
        } else {
            using LdsQuad = __attribute__((address_space(3))) shortx4;
            const char *p = lds + at[FI] + stage + PART * PLANE + S * 16 * 2 * ROWS;
            const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsQuad *)p);
            const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsQuad *)(p + 4 * 2 * ROWS));
            const u32x2 l = __builtin_bit_cast(u32x2, lo), h = __builtin_bit_cast(u32x2, hi);
            return u32x4{l.x, l.y, h.x, h.y};
        }
    }
};

__device__ __forceinline__ void mma_bf16(floatx16 &acc, const u32x4 &frag_n, const u32x4 &frag_m)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, frag_m), __builtin_bit_cast(bf16x8, frag_n), acc, 0, 0, 0);
}

// The same tile with the FP32 instructions, for operands that the parts cannot hold: the LDS layouts and fragments of mfma_kernel.h, two
// stages of 32 values of k, the next K-tile in registers, no pinned schedule.  la, lb: the operands' loaders, prepared; `aim_tile` aims at
// K-tile t (zeros past the end; tile 0 is the one that may lack values of k).
template <int BM, int BN, int NT, int FM, int FN, bool A_KCONTIG, bool B_KCONTIG, typename LoadA, typename LoadB, typename Aim>
__device__ __forceinline__ void exact_tile(floatx16 (&acc)[FN][FM], LoadA &la, LoadB &lb, char *lds, int ktiles, int first_ks, int wm0, int wn0,
                                           int thread, Aim &&aim_tile)
{
    constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
    const int lane = thread % 64;
    static_for<FM * FN>([&](auto X) { acc[decltype(X)::value / FM][decltype(X)::value % FM] = floatx16{}; });
    auto load = [&](int t) {
        __amdgpu_buffer_rsrc_t a, b;
        aim_tile(t, a, b);
        static_for<LoadA::LOADS>([&](auto Q) { la.template load<0, decltype(Q)::value>(a); });
        static_for<LoadB::LOADS>([&](auto Q) { lb.template load<0, decltype(Q)::value>(b); });
    };
    __syncthreads();                                   // every wavefront is done with the stages of the split parts
    if (ktiles > 0) load(0);
#pragma unroll 1
    for (int t = 0; t < ktiles; ++t) {
        char *stage = lds + (t & 1) * STAGE;
        if (t == 0) {
            static_for<LoadA::LOADS>([&](auto Q) { la.template cut<0, decltype(Q)::value>(first_ks, thread); });
            static_for<LoadB::LOADS>([&](auto Q) { lb.template cut<0, decltype(Q)::value>(first_ks, thread); });
        }
        la.store_floats(stage, thread);
        lb.store_floats(stage + A_BYTES, thread);
        load(t + 1);
        __syncthreads();                               // (the other stage is written only behind the next one)
#pragma unroll 1
        for (int step = 0; step < 4; ++step) {
            u32x4 a[FM], b[FN];
            static_for<FM>([&](auto F) { a[decltype(F)::value] = LoadA::read_floats(stage, lane, wm0, decltype(F)::value, step); });
            static_for<FN>([&](auto F) { b[decltype(F)::value] = LoadB::read_floats(stage + A_BYTES, lane, wn0, decltype(F)::value, step); });
            static_for<FM * FN>([&](auto X) {
                constexpr int i = decltype(X)::value % FM, j = decltype(X)::value / FM;
                mma(acc[j][i], b[j], a[i], float{});
            });
        }
    }
    __syncthreads();
}

template <int BM, int BN, int WM, int WN, bool A_KCONTIG, bool B_KCONTIG, bool EDGE, int DEPTH>
__global__ __launch_bounds__(WM *WN * 64, 2) void mfma_split_kernel(const MfmaArgs args)
{
    constexpr int NT = WM * WN * 64, BK = 32;
    constexpr int WTM = BM / WM, WTN = BN / WN, FM = WTM / 32, FN = WTN / 32;
    constexpr int SLOTS = FM * FN;                      // MFMAs per product and K-step
    using LoadA = SplitLoader<BM, NT, A_KCONTIG, EDGE, DEPTH>;
    using LoadB = SplitLoader<BN, NT, B_KCONTIG, EDGE, DEPTH>;
    constexpr int STAGE = LoadA::STAGE + LoadB::STAGE;
    extern __shared__ __attribute__((aligned(16))) char lds[];

    if constexpr (EDGE) {                              // grid layers behind the K slices: the fringe rows and columns (fringe.h)
        if (static_cast<int>(blockIdx.z) >= args.slices) {
            const int g = (static_cast<int>(blockIdx.z) - args.slices) * static_cast<int>(gridDim.x) + static_cast<int>(blockIdx.x);
            if (g < args.fringe_groups * args.slices)
                fringe_group<NT, A_KCONTIG, B_KCONTIG>(args, g % args.fringe_groups, g / args.fringe_groups, lds);
            return;
        }
    }
    int tm, tn;
    if (args.shape == 0) tile_coords(blockIdx.x, args.tiles_m, args.tiles_n, args.group_m, tm, tn);
    else tile_coords_balanced(blockIdx.x, args.tiles_m, args.tiles_n, args.group_m, args.reversed != 0, args.shape == MG_SHAPE_C_UPPER, tm, tn);
    const int64_t m0 = static_cast<int64_t>(tm) * BM, n0 = static_cast<int64_t>(tn) * BN;
    int kb = blockIdx.z * args.k_per_split;
    int ke = (kb + args.k_per_split < args.k) ? kb + args.k_per_split : args.k;
    if (!narrow_to_shape<BM, BN, BK>(args.shape, m0, n0, kb, ke)) return;

    const float *__restrict__ A = static_cast<const float *>(args.A);
    const float *__restrict__ B = static_cast<const float *>(args.B);
    const int rows_a = static_cast<int>(args.m_main - m0 < BM ? args.m_main - m0 : BM);
    const int rows_b = static_cast<int>(args.n_main - n0 < BN ? args.n_main - n0 : BN);
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int wm = wave % WM, wn = wave / WM;

    floatx16 acc[FN][FM], small[FN][FM];
    static_for<SLOTS>([&](auto X) { small[decltype(X)::value / FM][decltype(X)::value % FM] = acc[decltype(X)::value / FM][decltype(X)::value % FM] = floatx16{}; });

    LoadA la;
    LoadB lb;
    la.prepare(args.lda, rows_a, threadIdx.x);
    lb.prepare(args.ldb, rows_b, threadIdx.x);
    SplitFragments<BM, A_KCONTIG, FM> ra;
    SplitFragments<BN, B_KCONTIG, FN> rb;
    ra.prepare(lane, wm * WTM, 0);
    rb.prepare(lane, wn * WTN, LoadA::STAGE);

    // Tile 0 is the end of the sum (1 to 32 values of k), the others are whole: only the prologue has to cut anything.
    const int ktiles = (ke - kb + BK - 1) / BK;
    const int whole = (ktiles - 1) * BK, first_ks = ke - kb - whole;
    __amdgpu_buffer_rsrc_t aim_a, aim_b;
    auto aim_tile = [&](int t) __attribute__((always_inline)) {
        const int l0 = t == 0 ? kb + whole : kb + (t - 1) * BK;
        const int ks = t == 0 ? first_ks : (t < ktiles ? BK : 0);
        aim_a = LoadA::aim(A, args.lda, m0, l0, rows_a, ks);
        aim_b = LoadB::aim(B, args.ldb, n0, l0, rows_b, ks);
    };

    // fragments: a1, b1 double-buffered, the other parts not (they are read again once their last product is done)
    u32x4 a1[2][FM], b1[2][FN], a2[FM], a3[FM], b2[FN], b3[FN];
    auto read_first = [&](auto S, auto BUF, int stage, auto O) {      // O: which of the FM + FN reads
        constexpr int s = decltype(S)::value, buf = decltype(BUF)::value, o = decltype(O)::value;
        if constexpr (o < FM) a1[buf][o] = ra.template read<s, o, 0>(lds, stage);
        else b1[buf][o - FM] = rb.template read<s, o - FM, 0>(lds, stage);
    };
    auto read_second = [&](auto S, int stage, auto O) __attribute__((always_inline)) {
        constexpr int s = decltype(S)::value, o = decltype(O)::value;
        if constexpr (o < FM) a2[o] = ra.template read<s, o, 1>(lds, stage);
        else b2[o - FM] = rb.template read<s, o - FM, 1>(lds, stage);
    };
    auto read_third = [&](auto S, int stage, auto O) __attribute__((always_inline)) {
        constexpr int s = decltype(S)::value, o = decltype(O)::value;
        if constexpr (o < FM) a3[o] = ra.template read<s, o, 2>(lds, stage);
        else b3[o - FM] = rb.template read<s, o - FM, 2>(lds, stage);
    };
    constexpr int FRAGS = FM + FN;
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;

    // staging work of a K-tile: per piece the split of its two halves and its stores with the reload behind them
    constexpr int PIECES = LoadA::LOADS + LoadB::LOADS, EVENTS = 3 * PIECES;
    // one K-step: eight products of SLOTS MFMAs; the barrier of a K-tile sits in front of the seventh product of its last step
    constexpr int STEP_SLOTS = 8 * SLOTS, BARRIER_SLOT = STEP_SLOTS + 6 * SLOTS;
    auto event = [&](auto E, auto SET, int stage) __attribute__((always_inline)) {
        constexpr int e = decltype(E)::value, set = decltype(SET)::value;
        constexpr int piece = e / 3, w = e % 3;
        if constexpr (piece < LoadA::LOADS) {
            if constexpr (w < 2) la.template split<set, piece, w>();
            else { la.template store<piece>(lds + stage); la.template load<set, piece>(aim_a); }
        } else {
            constexpr int q = piece - LoadA::LOADS;
            if constexpr (w < 2) lb.template split<set, q, w>();
            else { lb.template store<q>(lds + LoadA::STAGE + stage); lb.template load<set, q>(aim_b); }
        }
    };

    // K-tile t from LDS stage CUR; the staged tile t + 1 (register set SET) goes to the other stage and its registers are
    // reloaded with tile t + 1 + DEPTH
    auto tile_body = [&](auto CUR, auto SET, int t) __attribute__((always_inline)) {
        constexpr int cur = decltype(CUR)::value * STAGE, nxt = (1 - decltype(CUR)::value) * STAGE;
        aim_tile(t + 1 + DEPTH);
        static_for<2>([&](auto S) __attribute__((always_inline)) {
            constexpr int s = decltype(S)::value;
            static_for<STEP_SLOTS>([&](auto G) __attribute__((always_inline)) {
                constexpr int g = decltype(G)::value, product = g / SLOTS, q = g % SLOTS, i = q % FM, j = q / FM;
                constexpr int tile_slot = s * STEP_SLOTS + g;
                if constexpr (tile_slot == BARRIER_SLOT) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                    __builtin_amdgcn_s_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                }
                if constexpr (product == 0) mma_bf16(small[j][i], b1[s][j], a3[i]);
                else if constexpr (product == 1) mma_bf16(small[j][i], b3[j], a1[s][i]);
                else if constexpr (product == 2) mma_bf16(small[j][i], b2[j], a3[i]);
                else if constexpr (product == 3) mma_bf16(small[j][i], b3[j], a2[i]);
                else if constexpr (product == 4) mma_bf16(small[j][i], b2[j], a2[i]);
                else if constexpr (product == 5) mma_bf16(small[j][i], b2[j], a1[s][i]);
                else if constexpr (product == 6) mma_bf16(small[j][i], b1[s][j], a2[i]);
                else mma_bf16(acc[j][i], b1[s][j], a1[s][i]);
                // reads for the next K-step: leading parts during the first four products, third parts during the fifth and sixth
                // (behind the barrier both during the seventh), second parts during the last
                auto spread = [&](auto slot0, auto slots, auto &&read) __attribute__((always_inline)) {
                    constexpr int z = g - decltype(slot0)::value, n = decltype(slots)::value;
                    if constexpr (z >= 0 && z < n)
                        static_for<share_begin(z + 1, FRAGS, n) - share_begin(z, FRAGS, n)>([&](auto R) {
                            read(std::integral_constant<int, share_begin(z, FRAGS, n) + decltype(R)::value>{});
                        });
                };
                using N1 = std::integral_constant<int, SLOTS>;
                using N2 = std::integral_constant<int, 2 * SLOTS>;
                using N4 = std::integral_constant<int, 4 * SLOTS>;
                using Seventh = std::integral_constant<int, 6 * SLOTS>;
                using Last = std::integral_constant<int, 7 * SLOTS>;
                if constexpr (s == 0) {
                    spread(C0{}, N4{}, [&](auto O) { read_first(C1{}, C1{}, cur, O); });
                    spread(N4{}, N2{}, [&](auto O) { read_third(C1{}, cur, O); });
                    spread(Last{}, N1{}, [&](auto O) { read_second(C1{}, cur, O); });
                } else {
                    spread(Seventh{}, N1{}, [&](auto O) { read_first(C0{}, C0{}, nxt, O); });
                    spread(Seventh{}, N1{}, [&](auto O) { read_third(C0{}, nxt, O); });
                    spread(Last{}, N1{}, [&](auto O) { read_second(C0{}, nxt, O); });
                }
                if constexpr (tile_slot < BARRIER_SLOT) {
                    static_for<share_begin(tile_slot + 1, EVENTS, BARRIER_SLOT) - share_begin(tile_slot, EVENTS, BARRIER_SLOT)>([&](auto R) {
                        event(std::integral_constant<int, share_begin(tile_slot, EVENTS, BARRIER_SLOT) + decltype(R)::value>{}, SET, nxt);
                    });
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };

    if (ktiles > 0) {
        // prologue: tile 0 -> LDS stage 0, tiles 1 .. DEPTH -> registers, first fragments.  Tile u sits in set u % DEPTH.
        aim_tile(0);
        static_for<LoadA::LOADS>([&](auto Q) { la.template load<0, decltype(Q)::value>(aim_a); });
        static_for<LoadB::LOADS>([&](auto Q) { lb.template load<0, decltype(Q)::value>(aim_b); });
        static_for<DEPTH - 1>([&](auto D) {
            constexpr int d = decltype(D)::value + 1;
            aim_tile(d);
            static_for<LoadA::LOADS>([&](auto Q) { la.template load<d, decltype(Q)::value>(aim_a); });
            static_for<LoadB::LOADS>([&](auto Q) { lb.template load<d, decltype(Q)::value>(aim_b); });
        });
        aim_tile(DEPTH);
        static_for<LoadA::LOADS>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            la.template cut<0, q>(first_ks, threadIdx.x);
            la.template split<0, q, 0>();
            la.template split<0, q, 1>();
            la.template store<q>(lds);
            la.template load<0, q>(aim_a);
        });
        static_for<LoadB::LOADS>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            lb.template cut<0, q>(first_ks, threadIdx.x);
            lb.template split<0, q, 0>();
            lb.template split<0, q, 1>();
            lb.template store<q>(lds + LoadA::STAGE);
            lb.template load<0, q>(aim_b);
        });
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        static_for<FRAGS>([&](auto O) { read_first(C0{}, C0{}, 0, O); });
        static_for<FRAGS>([&](auto O) { read_third(C0{}, 0, O); });
        static_for<FRAGS>([&](auto O) { read_second(C0{}, 0, O); });
    }
    constexpr int UNROLL = DEPTH > 2 ? DEPTH : 2;
    // After 8 K-tiles of a long sum and every 32 the wavefronts agree whether one of them has met an element that the parts cannot hold:
    // the rest of the sum would be for nothing (4096^3 of NaN 1596 -> 1084 us, FP32 pipes 916).
    bool given_up = false;
    int t = 0;
    for (;;) {
        const int next = t == 0 && ktiles > 32 ? 8 : t + 32, stop = next < ktiles ? next : ktiles;
        for (; t + UNROLL <= stop; t += UNROLL)
            static_for<UNROLL>([&](auto U) __attribute__((always_inline)) {
                constexpr int u = decltype(U)::value;
                tile_body(std::integral_constant<int, u % 2>{}, std::integral_constant<int, (u + 1) % DEPTH>{}, t + u);
            });
        if (t + UNROLL > ktiles) break;
        given_up = __syncthreads_or(la.beyond || lb.beyond);
        if (given_up) break;
    }
    if (!given_up)
        static_for<UNROLL - 1>([&](auto U) __attribute__((always_inline)) {
            constexpr int u = decltype(U)::value;
            if (t + u < ktiles) tile_body(std::integral_constant<int, u % 2>{}, std::integral_constant<int, (u + 1) % DEPTH>{}, t + u);
        });

    static_for<SLOTS>([&](auto X) { acc[decltype(X)::value / FM][decltype(X)::value % FM] += small[decltype(X)::value / FM][decltype(X)::value % FM]; });
    float watch = 0.f;                                 // becomes NaN when a sum is Inf or NaN
    if (!given_up)
        static_for<16 * SLOTS>([&](auto X) {
            constexpr int i = decltype(X)::value / 16 % FM, j = decltype(X)::value / 16 / FM;
            watch = fmaf(acc[j][i][decltype(X)::value % 16], 0.f, watch);
        });
    const bool redo = given_up || watch != 0.f;        // (an element beyond the parts leaves Inf or NaN in its sums)
    static_for<SLOTS>([&](auto X) { acc[decltype(X)::value / FM][decltype(X)::value % FM] *= SPLIT_UNSCALE; });
    // (what follows derives its lane numbers anew: kept through the K loop they would cost it registers)
    int thread = threadIdx.x;
    asm volatile("" : "+v"(thread));
    const int last_wave = thread / 64, last_wm = last_wave % WM, last_wn = last_wave / WM;
    if (__syncthreads_or(redo)) {                      // (also: every wavefront is done reading the operand stages)
        SplitLoader<BM, NT, A_KCONTIG, EDGE, 1> ea;
        SplitLoader<BN, NT, B_KCONTIG, EDGE, 1> eb;
        ea.prepare(args.lda, rows_a, thread);
        eb.prepare(args.ldb, rows_b, thread);
        exact_tile<BM, BN, NT, FM, FN, A_KCONTIG, B_KCONTIG>(acc, ea, eb, lds, ktiles, first_ks, last_wm * WTM, last_wn * WTN, thread,
                                                             [&](int t_, __amdgpu_buffer_rsrc_t &a, __amdgpu_buffer_rsrc_t &b) { aim_tile(t_); a = aim_a; b = aim_b; });
    }
    tile_epilogue<float, 32, FM, FN, WTM, WTN, EDGE>(acc, args, lds, m0, n0, last_wm, last_wn, last_wave, thread % 64);
}

}  // namespace mg
