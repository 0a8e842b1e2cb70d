// FP32 macro-tile GEMM kernel on the bf16 matrix pipes.
//
// Every FP32 element is the sum of three bf16 values, x = x1 + x2 + x3 (each the rounded rest of the one before: 3 x 8
// significand bits and their signs hold all 24), and of the nine products of two such elements the six that matter are
// taken:  a1 b1 + (a1 b2 + a2 b1 + a2 b2 + a1 b3 + a3 b1); the rest is below 2^-26 of |a b|, a quarter of what rounding
// a b to FP32 costs.  Products of bf16 values are exact in the matrix pipes' FP32 accumulators; a1 b1 has accumulators of its own, the five
// small products share others that are added once at the end, so the large sums see one rounding per four values of k
// (v_mfma_f32_32x32x16_bf16) where v_mfma_f32_32x32x2_f32 rounds for each.  Six bf16 instructions of 32 cycles take the
// place of eight FP32 ones of 64 (16 values of k).
//
// The sums differ from FP32 arithmetic where a part cannot hold its share: elements below 2^-110 (but not 0), whose last bits lie
// below bf16's smallest value, and elements or products near the end of the range, which leave Inf or NaN in an
// accumulator.  The kernel watches for both (the rest that the third part rounds is 0 or at least 2^(e - 23) for an element of exponent e and at most
// 2^(e - 17): subnormal whenever bits are lost; a test of the sums) and a work-group that meets either computes its
// tile again with the FP32 instructions.
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

// two elements -> their three parts, packed
struct SplitPair {
    uint32_t part[3];
};
__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{a, b}), bf16x2));
}
// (tiny: set when bits may have been lost below bf16's range, the rest that the third part rounds being subnormal)
__device__ __forceinline__ SplitPair split_pair(float a, float b, bool &tiny)
{
    SplitPair s;
    s.part[0] = bf16_pair(a, b);
    a -= __builtin_bit_cast(float, s.part[0] << 16);
    b -= __builtin_bit_cast(float, s.part[0] & 0xffff0000u);
    s.part[1] = bf16_pair(a, b);
    a -= __builtin_bit_cast(float, s.part[1] << 16);
    b -= __builtin_bit_cast(float, s.part[1] & 0xffff0000u);
    s.part[2] = bf16_pair(a, b);
    constexpr int SUBNORMAL = 0x90;
    tiny |= __builtin_amdgcn_classf(a, SUBNORMAL) | __builtin_amdgcn_classf(b, SUBNORMAL);
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
    static constexpr uint32_t OUT_OF_RANGE = 0x80000000u;

    u32x4 regs[DEPTH][LOADS];
    uint32_t goff[LOADS];
    int slot[LOADS];                // LDS byte offset of each piece inside a plane
    bool keep[4];                   // EDGE, along the rows: element e of this lane's pieces is a row that exists
    bool tiny;                      // see split_pair
    SplitPair made[2];              // the piece being split

    __device__ __forceinline__ void prepare(int64_t ld, int rows, int t)
    {
        tiny = false;
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
                slot[Q] = ldsmap::split_line_slot(ROWS, l, mc / 2) + 8 * (mc % 2);
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
        made[HALF] = split_pair(v[0], v[1], tiny);
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
// K-tile t (zeros past the end; tile 0 is the one that may lack values of k).  multiplies: the same for a whole wavefront; false: it
// only loads.
template <int BM, int BN, int NT, int FM, int FN, bool A_KCONTIG, bool B_KCONTIG, typename LoadA, typename LoadB, typename Aim>
__device__ __forceinline__ void exact_tile(floatx16 (&acc)[FN][FM], LoadA &la, LoadB &lb, char *lds, int ktiles, int first_ks, int wm0, int wn0,
                                           int thread, Aim &&aim_tile, bool multiplies = true)
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
        for (int step = multiplies ? 0 : 4; step < 4; ++step) {
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
    // one K-step: six products of SLOTS MFMAs; the barrier of a K-tile sits in front of the fifth product of its last step
    constexpr int STEP_SLOTS = 6 * SLOTS, BARRIER_SLOT = STEP_SLOTS + 4 * SLOTS;
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
                else if constexpr (product == 2) mma_bf16(small[j][i], b2[j], a2[i]);
                else if constexpr (product == 3) mma_bf16(small[j][i], b2[j], a1[s][i]);
                else if constexpr (product == 4) mma_bf16(small[j][i], b1[s][j], a2[i]);
                else mma_bf16(acc[j][i], b1[s][j], a1[s][i]);
                // reads for the next K-step: leading parts during the first two products, third parts during the next
                // two (behind the barrier both during the fifth), second parts during the last
                auto spread = [&](auto slot0, auto slots, auto &&read) __attribute__((always_inline)) {
                    constexpr int z = g - decltype(slot0)::value, n = decltype(slots)::value;
                    if constexpr (z >= 0 && z < n)
                        static_for<share_begin(z + 1, FRAGS, n) - share_begin(z, FRAGS, n)>([&](auto R) {
                            read(std::integral_constant<int, share_begin(z, FRAGS, n) + decltype(R)::value>{});
                        });
                };
                using N1 = std::integral_constant<int, SLOTS>;
                using N2 = std::integral_constant<int, 2 * SLOTS>;
                if constexpr (s == 0) {
                    spread(C0{}, N2{}, [&](auto O) { read_first(C1{}, C1{}, cur, O); });
                    spread(std::integral_constant<int, 2 * SLOTS>{}, N2{}, [&](auto O) { read_third(C1{}, cur, O); });
                    spread(std::integral_constant<int, 5 * SLOTS>{}, N1{}, [&](auto O) { read_second(C1{}, cur, O); });
                } else {
                    spread(std::integral_constant<int, 4 * SLOTS>{}, N1{}, [&](auto O) { read_first(C0{}, C0{}, nxt, O); });
                    spread(std::integral_constant<int, 4 * SLOTS>{}, N1{}, [&](auto O) { read_third(C0{}, nxt, O); });
                    spread(std::integral_constant<int, 5 * SLOTS>{}, N1{}, [&](auto O) { read_second(C0{}, nxt, O); });
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
    // Every 32 K-tiles the wavefronts agree whether one of them has met an element that the parts cannot hold: the rest of the
    // sum would be for nothing.
    bool given_up = false;
    int t = 0;
    for (;;) {
        const int stop = t + 32 < ktiles ? t + 32 : ktiles;
        for (; t + UNROLL <= stop; t += UNROLL)
            static_for<UNROLL>([&](auto U) __attribute__((always_inline)) {
                constexpr int u = decltype(U)::value;
                tile_body(std::integral_constant<int, u % 2>{}, std::integral_constant<int, (u + 1) % DEPTH>{}, t + u);
            });
        if (t + UNROLL > ktiles) break;
        given_up = __syncthreads_or(la.tiny || lb.tiny);
        if (given_up) break;
    }
    if (!given_up)
        static_for<UNROLL - 1>([&](auto U) __attribute__((always_inline)) {
            constexpr int u = decltype(U)::value;
            if (t + u < ktiles) tile_body(std::integral_constant<int, u % 2>{}, std::integral_constant<int, (u + 1) % DEPTH>{}, t + u);
        });

    float watch = 0.f;                                 // becomes NaN when a sum is Inf or NaN
    static_for<SLOTS>([&](auto X) {
        constexpr int i = decltype(X)::value % FM, j = decltype(X)::value / FM;
        acc[j][i] += small[j][i];
        static_for<16>([&](auto R) { watch = fmaf(acc[j][i][decltype(R)::value], 0.f, watch); });
    });
    const bool redo = given_up || la.tiny || lb.tiny || watch != 0.f;
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

// 64 x 64 tiles of grids that leave a compute unit one or two of them: no barrier in the K loop.  Each of the eight
// wavefronts holds the whole tile and takes every eighth slice of 16 values of k, so that no element is loaded or split
// twice; a slice goes from memory through registers to the wavefront's own part of LDS (coalesced 16-byte pieces in, MFMA operand layout
// out: operands along k loaded in that layout directly cost a clock per lane), is read a fragment at a time, split, and multiplied while the next
// one is split.  The eight sums meet in LDS at the end.  (The tile cut among wavefronts that share their fragments
// reads 9 fragments from LDS for 6 MFMAs, this one 12 for 24.)  One set of accumulators: an eighth of the sum each, and the products
// of a slice added smallest first, still round less than FP32 instructions do.
template <bool KCONTIG, bool EDGE> struct SliceLoader {
    static constexpr int PIECES = 4;                   // 16-byte pieces per lane and slice (64 rows x 16 values of k)
    static constexpr int BYTES = 4096;
    using Set = u32x4[PIECES];
    Set regs;
    uint32_t goff[PIECES];
    uint32_t keep[4];              // EDGE, along the rows: all ones where element e of this lane's pieces is a row that exists
    int slot[2], at[2];            // LDS: where pieces 0, 1 | 2, 3 go, where the values of fragment 0 | 1 are
    u32x4 raw[2][2];               // fragments read back, two at a time: 8 values each
    bool tiny;                     // see split_pair

    __device__ __forceinline__ void prepare(int64_t ld, int rows, int lane, int offset)
    {
        tiny = false;
        static_for<PIECES>([&](auto Qc) {
            constexpr int q = decltype(Qc)::value;
            if constexpr (KCONTIG) goff[q] = static_cast<uint32_t>(((16 * q + lane / 4) * ld + lane % 4 * 4) * 4);
            else goff[q] = !EDGE || lane % 16 * 4 < rows ? static_cast<uint32_t>(((4 * q + lane / 16) * ld + lane % 16 * 4) * 4) : 0x80000000u;
        });
#pragma unroll
        for (int e = 0; e < 4; ++e) keep[e] = !EDGE || KCONTIG || lane % 16 * 4 + e < rows ? ~0u : 0u;
        if constexpr (KCONTIG) {
            slot[0] = slot[1] = offset + ldsmap::split_row_slot(lane / 4, lane % 4);
            at[0] = offset + ldsmap::split_row_slot(lane % 32, 2 * (lane / 32));
            at[1] = at[0] ^ 16;                        // (the other half of the lane's 8 values)
        } else {
            slot[0] = offset + ldsmap::slice_line_slot(lane / 16, lane % 16);
            slot[1] = offset + ldsmap::slice_line_slot(8 + lane / 16, lane % 16) - 2048;
            at[0] = offset + ldsmap::slice_line_slot(8 * (lane / 32), lane % 32 / 4) + lane % 4 * 4;
            at[1] = offset + ldsmap::slice_line_slot(8 * (lane / 32), 8 + lane % 32 / 4) + lane % 4 * 4;
        }
    }
    // ks <= 16 values of k from l0 on (ks <= 0: zeros, no access); the descriptor ends with the last element that exists
    __device__ __forceinline__ static __amdgpu_buffer_rsrc_t aim(const float *X, int64_t ld, int64_t r0, int64_t l0, int rows, int ks)
    {
        const float *base = KCONTIG ? X + r0 * ld + l0 : X + r0 + l0 * ld;
        if (ks > 16) ks = 16;
        const int64_t extent = KCONTIG ? (rows - 1) * ld + ks : (ks - 1) * ld + rows;
        const int range = static_cast<int>(extent * 4) & -static_cast<int>(ks > 0);      // (no branch: it would cut the K loop's schedule)
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, range, 0x00020000);
    }
    template <int Q> __device__ __forceinline__ void load(Set &set, __amdgpu_buffer_rsrc_t rsrc) const
    {
        set[Q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, goff[Q], 0, 0);
    }
    // operand along k: values beyond the sum are the next row's
    __device__ __forceinline__ void cut(int ks, int lane)
    {
        if constexpr (KCONTIG)
            static_for<16>([&](auto X) {
                constexpr int q = decltype(X)::value / 4, e = decltype(X)::value % 4;
                regs[q][e] = lane % 4 * 4 + e < ks ? regs[q][e] : 0u;
            });
    }
    template <int Q> __device__ __forceinline__ void store(const Set &set, char *buffer) const
    {
        u32x4 v = set[Q];
        if constexpr (EDGE && !KCONTIG) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] &= keep[e];
        }
        *reinterpret_cast<u32x4 *>(buffer + slot[Q / 2] + Q * 1024) = v;
    }
    // fragment F of the slice in `buffer` -> raw[F]
    template <int F> __device__ __forceinline__ void read(const char *buffer)
    {
        if constexpr (KCONTIG) {
            raw[F][0] = *reinterpret_cast<const u32x4 *>(buffer + at[0] + F * 2048);
            raw[F][1] = *reinterpret_cast<const u32x4 *>(buffer + at[1] + F * 2048);
        } else {
            static_for<8>([&](auto E) {
                constexpr int e = decltype(E)::value;
                raw[F][e / 4][e % 4] = *reinterpret_cast<const uint32_t *>(buffer + at[F] + e * 256);
            });
        }
    }
    // values 2 PAIR and 2 PAIR + 1 of fragment F -> their three parts
    template <int F, int PAIR> __device__ __forceinline__ void split(u32x4 (&part)[3])
    {
        const uint32_t x = raw[F][PAIR / 2][2 * (PAIR % 2)], y = raw[F][PAIR / 2][2 * (PAIR % 2) + 1];
        const SplitPair s = split_pair(__builtin_bit_cast(float, x), __builtin_bit_cast(float, y), tiny);
        part[0][PAIR] = s.part[0];
        part[1][PAIR] = s.part[1];
        part[2][PAIR] = s.part[2];
    }
};

template <bool A_KCONTIG, bool B_KCONTIG, bool EDGE>
__global__ __launch_bounds__(512, 2) void mfma_split_slices_kernel(const MfmaArgs args)
{
    constexpr int BM = 64, BN = 64, WAVES = 8, NT = 512, SLICE = 16;
    constexpr int ROWB = BM * 4 + 16, REGION = BN * ROWB;      // one wavefront's sums: [column][row] floats
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
    if (!narrow_to_shape<BM, BN, 32>(args.shape, m0, n0, kb, ke)) return;

    const float *__restrict__ A = static_cast<const float *>(args.A);
    const float *__restrict__ B = static_cast<const float *>(args.B);
    const int rows_a = static_cast<int>(args.m_main - m0 < BM ? args.m_main - m0 : BM);
    const int rows_b = static_cast<int>(args.n_main - n0 < BN ? args.n_main - n0 : BN);
    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);

    floatx16 acc[2][2];
    static_for<4>([&](auto X) { acc[decltype(X)::value / 2][decltype(X)::value % 2] = floatx16{}; });
    SliceLoader<A_KCONTIG, EDGE> la;
    SliceLoader<B_KCONTIG, EDGE> lb;
    constexpr int BUFFER = SliceLoader<A_KCONTIG, EDGE>::BYTES + SliceLoader<B_KCONTIG, EDGE>::BYTES;     // one slice
    static_assert(2 * BUFFER * WAVES <= WAVES * REGION, "two slices per wavefront");
    la.prepare(args.lda, rows_a, lane, wave * 2 * BUFFER);
    lb.prepare(args.ldb, rows_b, lane, wave * 2 * BUFFER + SliceLoader<A_KCONTIG, EDGE>::BYTES);

    // rounds of eight slices, the last (which may lack values of k, or whole slices) first
    const int rounds = (ke - kb + WAVES * SLICE - 1) / (WAVES * SLICE);
    __amdgpu_buffer_rsrc_t aim_a, aim_b;
    auto aim_round = [&](int u) __attribute__((always_inline)) {
        const int l0 = kb + ((rounds - 1 - u) * WAVES + wave) * SLICE, ks = u < rounds ? ke - l0 : 0;
        aim_a = la.aim(A, args.lda, m0, l0, rows_a, ks);
        aim_b = lb.aim(B, args.ldb, n0, l0, rows_b, ks);
    };
    u32x4 a[2][2][3], b[2][2][3];                      // buffer, fragment, part
    // fragments in the order a0 b0 a1 b1: F of the slice in LDS buffer BUF -> raw registers; four pairs each -> parts
    auto read = [&](auto F, auto BUF) __attribute__((always_inline)) {
        constexpr int f = decltype(F)::value;
        const char *buffer = lds + decltype(BUF)::value * BUFFER;
        if constexpr (f % 2 == 0) la.template read<f / 2>(buffer);
        else lb.template read<f / 2>(buffer);
    };
    auto split = [&](auto E, auto BUF) __attribute__((always_inline)) {
        constexpr int e = decltype(E)::value, f = e / 8, pair = e % 4, buf = decltype(BUF)::value;
        if constexpr (e / 4 % 2 == 0) la.template split<f, pair>(a[buf][f]);
        else lb.template split<f, pair>(b[buf][f]);
    };
    // piece Q (0 .. 7) of a staged slice -> LDS buffer BUF, and its registers loaded again
    auto store = [&](auto Q, auto BUF) __attribute__((always_inline)) {
        constexpr int q = decltype(Q)::value / 2;
        char *buffer = lds + decltype(BUF)::value * BUFFER;
        if constexpr (decltype(Q)::value % 2 == 0) { la.template store<q>(la.regs, buffer); la.template load<q>(la.regs, aim_a); }
        else { lb.template store<q>(lb.regs, buffer); lb.template load<q>(lb.regs, aim_b); }
    };
    // Slice u from fragment buffer BUF, the smallest products first.  MORE: meanwhile slice u + 1 is split into the other buffer (its first
    // fragment has been read, the others are read six MFMAs ahead), slice u + 2 goes to LDS, u + 3 is asked for.
    auto multiply = [&](auto BUF, auto MORE) __attribute__((always_inline)) {
        constexpr int buf = decltype(BUF)::value;
        using Mine = std::integral_constant<int, buf>;
        using Other = std::integral_constant<int, 1 - buf>;
        constexpr int pb[6] = {0, 2, 1, 1, 0, 0}, pa[6] = {2, 0, 1, 0, 1, 0};
        static_for<24>([&](auto X) __attribute__((always_inline)) {
            constexpr int x = decltype(X)::value, p = x / 4, i = x % 2, j = x / 2 % 2;
            mma_bf16(acc[j][i], b[buf][j][pb[p]], a[buf][i][pa[p]]);
            if constexpr (decltype(MORE)::value) {
                if constexpr (x % 6 == 0 && x < 18) read(std::integral_constant<int, x / 6 + 1>{}, Other{});
                if constexpr (x == 18) read(std::integral_constant<int, 0>{}, Mine{});
                if constexpr (x % 2 == 0 && x < 16) store(std::integral_constant<int, x / 2>{}, Mine{});
                static_for<share_begin(x + 1, 16, 24) - share_begin(x, 16, 24)>([&](auto R) __attribute__((always_inline)) {
                    split(std::integral_constant<int, share_begin(x, 16, 24) + decltype(R)::value>{}, Other{});
                });
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    };
    // eight columns of C per wavefront, four at a time: four consecutive rows of a column per lane; the old values of whole pieces
    // are asked for before the sum
    const int row = lane % 16 * 4, col = wave * 8 + lane / 16;
    const bool held = args.beta != 0.f && args.partial == nullptr && args.mask == 0;
    floatx4 old[2];
    auto piece_left = [&](int pass) __attribute__((always_inline)) {
        const int64_t left = args.m_main - m0 - row;
        return n0 + col + 4 * pass >= args.n_main || left <= 0 ? 0 : (left < 4 ? static_cast<int>(left) : 4);
    };
    static_for<2>([&](auto P) {
        constexpr int pass = decltype(P)::value;
        old[pass] = floatx4{};
        if (held && piece_left(pass) == 4) {
            const auto v = *reinterpret_cast<const Pack<float, 4> *>(static_cast<const float *>(args.C) + m0 + row + (n0 + col + 4 * pass) * args.ldc);
            old[pass] = floatx4{v.v[0], v.v[1], v.v[2], v.v[3]};
        }
    });
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    if (rounds > 0) {
        typename SliceLoader<A_KCONTIG, EDGE>::Set second_a;
        typename SliceLoader<B_KCONTIG, EDGE>::Set second_b;
        aim_round(0);
        static_for<4>([&](auto Q) { la.template load<decltype(Q)::value>(la.regs, aim_a); lb.template load<decltype(Q)::value>(lb.regs, aim_b); });
        aim_round(1);
        static_for<4>([&](auto Q) { la.template load<decltype(Q)::value>(second_a, aim_a); lb.template load<decltype(Q)::value>(second_b, aim_b); });
        aim_round(2);
        const int ks = ke - (kb + ((rounds - 1) * WAVES + wave) * SLICE);
        la.cut(ks, lane);
        lb.cut(ks, lane);
        static_for<8>([&](auto Q) { store(Q, C0{}); });
        static_for<4>([&](auto F) { read(F, C0{}); });
        static_for<16>([&](auto E) { split(E, C0{}); });
        static_for<4>([&](auto Q) { la.template store<decltype(Q)::value>(second_a, lds + BUFFER); lb.template store<decltype(Q)::value>(second_b, lds + BUFFER); });
        read(C0{}, C1{});
        int u = 0;
        for (; u + 2 < rounds; u += 2) {
            aim_round(u + 3);
            multiply(C0{}, std::true_type{});
            aim_round(u + 4);
            multiply(C1{}, std::true_type{});
        }
        if (u + 1 < rounds) {
            aim_round(rounds);
            multiply(C0{}, std::true_type{});
            multiply(C1{}, std::false_type{});
        } else {
            multiply(C0{}, std::false_type{});
        }
    }
    __syncthreads();                                   // the sums take the place of the slices

    char *mine = lds + wave * REGION;
    auto put = [&](char *region, const floatx16 &v, int row, int col) __attribute__((always_inline)) {
        static_for<4>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            *reinterpret_cast<floatx4 *>(region + (col + lane % 32) * ROWB + (row + 8 * q + 4 * (lane / 32)) * 4) =
                floatx4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        });
    };
    static_for<4>([&](auto X) {
        constexpr int i = decltype(X)::value % 2, j = decltype(X)::value / 2;
        put(mine, acc[j][i], 32 * i, 32 * j);
    });
    __syncthreads();
    floatx4 sum[2];
    float watch = 0.f;                                 // becomes NaN when a sum is Inf or NaN
    auto gather = [&](int regions) __attribute__((always_inline)) {
        static_for<2>([&](auto P) {
            constexpr int pass = decltype(P)::value;
            const char *p = lds + (col + 4 * pass) * ROWB + row * 4;
            sum[pass] = *reinterpret_cast<const floatx4 *>(p);
            for (int w = 1; w < regions; ++w) sum[pass] += *reinterpret_cast<const floatx4 *>(p + w * REGION);
        });
    };
    gather(WAVES);
    static_for<8>([&](auto E) { watch = fmaf(sum[decltype(E)::value / 4][decltype(E)::value % 4], 0.f, watch); });
    if (__syncthreads_or(la.tiny || lb.tiny || watch != 0.f)) {
        floatx16 exact[1][1];
        SplitLoader<BM, NT, A_KCONTIG, EDGE, 1> ea;
        SplitLoader<BN, NT, B_KCONTIG, EDGE, 1> eb;
        ea.prepare(args.lda, rows_a, threadIdx.x);
        eb.prepare(args.ldb, rows_b, threadIdx.x);
        const int ktiles = (ke - kb + 31) / 32, whole = (ktiles - 1) * 32;
        exact_tile<BM, BN, NT, 1, 1, A_KCONTIG, B_KCONTIG>(exact, ea, eb, lds, ktiles, ke - kb - whole, wave % 2 * 32, wave / 2 % 2 * 32, threadIdx.x,
                                                           [&](int t, __amdgpu_buffer_rsrc_t &x, __amdgpu_buffer_rsrc_t &y) {
                                                               const int l0 = t == 0 ? kb + whole : kb + (t - 1) * 32, ks = t < ktiles ? ke - l0 : 0;
                                                               x = ea.aim(A, args.lda, m0, l0, rows_a, ks);
                                                               y = eb.aim(B, args.ldb, n0, l0, rows_b, ks);
                                                           }, wave < 4);
        if (wave < 4) put(lds, exact[0][0], wave % 2 * 32, wave / 2 * 32);
        __syncthreads();
        gather(1);
    }
    static_for<2>([&](auto P) {
        constexpr int pass = decltype(P)::value;
        const int64_t gm = m0 + row, gn = n0 + col + 4 * pass;
        int first = 0, valid = piece_left(pass);
        if (args.mask != 0) {                          // as tile_epilogue: the wanted triangle of C
            const int64_t d = gn - gm;
            if (args.shape == MG_SHAPE_C_LOWER) first = d > 0 ? (d < 4 ? static_cast<int>(d) : 4) : 0;
            else valid = d + 1 < valid ? (d + 1 > 0 ? static_cast<int>(d + 1) : 0) : valid;
        }
        const bool raw = args.partial != nullptr;
        float *p = raw ? args.partial + (static_cast<int64_t>(blockIdx.z) * args.n + gn) * args.m + gm : static_cast<float *>(args.C) + gm + gn * args.ldc;
        const float alpha = raw ? 1.f : args.alpha, beta = raw ? 0.f : args.beta;
        if (first == 0 && valid == 4) {
            Pack<float, 4> o;
            if (beta != 0.f) {
                if (!held) {
                    const Pack<float, 4> c = *reinterpret_cast<const Pack<float, 4> *>(p);
                    old[pass] = floatx4{c.v[0], c.v[1], c.v[2], c.v[3]};
                }
                static_for<4>([&](auto E) { o.v[decltype(E)::value] = fmaf(beta, old[pass][decltype(E)::value], alpha * sum[pass][decltype(E)::value]); });
            } else {
                static_for<4>([&](auto E) { o.v[decltype(E)::value] = alpha * sum[pass][decltype(E)::value]; });
            }
            *reinterpret_cast<Pack<float, 4> *>(p) = o;
        } else {
            static_for<4>([&](auto E) {
                constexpr int e = decltype(E)::value;
                if (e >= first && e < valid) {
                    float o = alpha * sum[pass][e];
                    if (beta != 0.f) o = fmaf(beta, p[e], o);
                    p[e] = o;
                }
            });
        }
    });
}

}  // namespace mg
