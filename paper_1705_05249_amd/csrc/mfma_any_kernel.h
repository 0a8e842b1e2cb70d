// FP16 macro-tile GEMM kernel for operands whose rows start at any element and sizes that end anywhere: the tiles, LDS layouts and fragments of
// the direct-to-LDS kernel (mfma_dma_kernel.h), but every 16-byte piece passes through registers, where it may come from any element.
//
// What bounds it: what a compute unit's L1 passes on (a row of a tile that does not start on a line of the cache touches two lines for the
// data of one; 16-byte loads of rows of 128 bytes from the L2 on 256 compute units: 27 TB/s where rows start on lines, 16 where they do not, 15 at odd
// elements), latency (DEPTH K-tiles are in flight in registers), and, in calls of around ten microseconds, the instructions
// themselves, which a compute unit fetches at a few bytes per clock when it meets them for the first time.  So everything is there once: the end of the
// sum is a K-tile like the others, the first one, whose loads are as wide (see load_end); the unrolled loop is left from its middle
// instead of being followed by copies of its bodies; and the epilogue is one short loop over the tile in LDS.
//
// K-tiles: tile 0 is the end of the sum (1 to 64 values of k), all others are whole and loaded without checks:
//   * operand along k: lanes in missing rows read a row that exists;
//   * operand along its rows: a piece that straddles the last row runs into the next line, up to seven elements of it.  The line behind a
//     whole K-tile's last one belongs to the matrix (tile 0 has at least one), and eight rows or more keep the seven inside it; lanes
//     whose whole piece is missing read the line's first one.
// What such lanes put into LDS reaches rows and columns of C that do not exist.
#pragma once

#include "mfma_dma_kernel.h"

namespace mg {

// v moved down by `by` halves (8 and more: zeros), zeros from above
__device__ __forceinline__ u32x4 shift_down(u32x4 v, int by)
{
    if (by & 2) v = u32x4{v[1], v[2], v[3], 0u};
    if (by & 4) v = u32x4{v[2], v[3], 0u, 0u};
    if (by & 1) v = u32x4{v[0] >> 16 | v[1] << 16, v[1] >> 16 | v[2] << 16, v[2] >> 16 | v[3] << 16, v[3] >> 16};
    return by >= 8 ? u32x4{0u, 0u, 0u, 0u} : v;
}

// v moved down by `by` elements
template <typename T> __device__ __forceinline__ u32x4 shift_elements(u32x4 v, int by)
{
    return shift_down(v, sizeof(T) == 4 ? 2 * by : by);
}

// the first `valid` (1 to V - 1) elements of a piece: halves of the piece, of the rest, ...
template <typename T> __device__ __forceinline__ void store_first(T *out, const Pack<T, 16 / sizeof(T)> &o, int valid)
{
    const u32x4 w = __builtin_bit_cast(u32x4, o);
    if constexpr (sizeof(T) == 2) {
        if (valid & 4) *reinterpret_cast<Pack<T, 4> *>(out) = __builtin_bit_cast(Pack<T, 4>, u32x2{w.x, w.y});
        const uint32_t two = valid & 4 ? w.z : w.x, next = valid & 4 ? w.w : w.y;
        if (valid & 2) *reinterpret_cast<Pack<T, 2> *>(out + (valid & 4)) = __builtin_bit_cast(Pack<T, 2>, two);
        const uint16_t one = static_cast<uint16_t>(valid & 2 ? next : two);
        if (valid & 1) out[valid & 6] = __builtin_bit_cast(T, one);
    } else {
        if (valid & 2) *reinterpret_cast<Pack<T, 2> *>(out) = __builtin_bit_cast(Pack<T, 2>, u32x2{w.x, w.y});
        if (valid & 1) out[valid & 2] = __builtin_bit_cast(T, valid & 2 ? w.z : w.x);
    }
}

// One operand tile (ROWS rows x 64 k): global -> registers -> LDS
template <int ROWS, int NT, bool KCONTIG, int RB, int DEPTH> struct AnyLoader {
    static constexpr int LDS_BYTES = ROWS * 128;
    static constexpr int COUNT = LDS_BYTES / (NT * 16);                // 16-byte pieces per thread
    static constexpr int RCH = ROWS / 8;                               // pieces per line of an operand along its rows
    static_assert(COUNT >= 1 && COUNT * NT * 16 == LDS_BYTES, "tile / work-group size");

    u32x4 regs[DEPTH][COUNT];
    uint32_t goff[COUNT];      // byte offset of each piece from the tile's first element
    int slot[COUNT];           // and in LDS, from the operand stage's start
    const char *base;
    uint32_t lanes;            // all bits, or none: every lane loads the same 16 bytes

    __device__ __forceinline__ void prepare(int64_t ld, int rows, int t)
    {
        static_for<COUNT>([&](auto Qc) {
            constexpr int Q = decltype(Qc)::value;
            const int idx = t + Q * NT;
            if constexpr (KCONTIG) {
                const int r = idx / 8, c = idx % 8;
                goff[Q] = static_cast<uint32_t>(((r < rows ? r : rows - 1) * ld + c * 8) * 2);
                slot[Q] = ldsmap::kcontig_slot<RB>(r, c);
            } else {
                const int l = idx / RCH, c = idx % RCH;
                goff[Q] = static_cast<uint32_t>((l * ld + (c * 8 < rows ? c * 8 : 0)) * 2);
                slot[Q] = ldsmap::transposed_slot(ROWS, l, c);
            }
        });
    }
    // exists: else a tile past the end of the sum, whose loads (into registers nobody stores) all take the first 16 bytes at l0
    __device__ __forceinline__ void aim(const _Float16 *X, int64_t ld, int64_t r0, int64_t l0, bool exists)
    {
        base = reinterpret_cast<const char *>(KCONTIG ? X + r0 * ld + l0 : X + r0 + l0 * ld);
        lanes = exists ? ~0u : 0u;
    }
    template <int SET, int Q> __device__ __forceinline__ void load()
    {
        uint32_t at = goff[Q] & lanes;
        // (scalar base + 32-bit lane offset; without this line the offsets are widened in front of the K loop)
        asm volatile("" : "+v"(at));
        regs[SET][Q] = load_unaligned_chunk<_Float16>(reinterpret_cast<const _Float16 *>(base + at));
    }
    // Of the K-tile of `ks` values of k that ends with the sum (and may hold the matrix's last line): a piece that ends beyond its line is
    // loaded as the 16 bytes that end with the line, which has eight elements or more, and moved down when it is stored (cut).
    static __device__ __forceinline__ int back(int rows, int ks, int idx)
    {
        const int beyond = KCONTIG ? idx % 8 * 8 + 8 - ks : idx % RCH * 8 + 8 - rows;
        return beyond > 0 ? beyond : 0;
    }
    template <int SET, int Q> __device__ __forceinline__ void load_end(int64_t ld, int rows, int ks, int t)
    {
        const int idx = t + Q * NT, r = idx / 8, l = idx / RCH;
        const int64_t at = KCONTIG ? (r < rows ? r : rows - 1) * ld + idx % 8 * 8 : (l < ks ? l : ks - 1) * ld + idx % RCH * 8;
        regs[SET][Q] = load_unaligned_chunk<_Float16>(reinterpret_cast<const _Float16 *>(base) + at - back(rows, ks, idx));
    }
    template <int SET, int Q> __device__ __forceinline__ void cut(int rows, int ks, int t)
    {
        const int idx = t + Q * NT;
        regs[SET][Q] = shift_down(regs[SET][Q], KCONTIG || idx / RCH < ks ? back(rows, ks, idx) : 8);
    }
    template <int SET, int Q> __device__ __forceinline__ void store(char *stage) const
    {
        *reinterpret_cast<u32x4 *>(stage + slot[Q]) = regs[SET][Q];
    }
};

#if defined(__HIP_DEVICE_COMPILE__)
// MFMA operand of fragment F, K-step S, from an operand stage at byte offset STAGE (read_operand of mfma_dma_kernel.h, as reads that the
// compiler waits for)
template <bool KCONTIG, int ROWS, int F, int RB, int S, int STAGE> __device__ __forceinline__ u32x4 read_tracked(lds_char *lds3, const int (&frag)[8])
{
    if constexpr (KCONTIG) {
        return *reinterpret_cast<const __attribute__((address_space(3))) u32x4 *>(lds3 + frag[frag_select<RB>(F, S)] + F * RB * 128 + STAGE);
    } else {
        constexpr int LINE = 2 * ROWS;
        lds_char *p = lds3 + frag[F] + S * ((512 / RB) * LINE) + STAGE;
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)p);
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)(p + 4 * LINE));
        return __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
}
#endif

// The tile's results through LDS: [column][m] floats of the whole tile, then every thread takes 16-byte pieces of C (or of the partial sums),
// consecutive threads consecutive pieces of a column, so that a wavefront's stores are whole columns of the tile.
// 16 x 16 blocks: lane l holds rows 4 (l / 16) .. + 3 of column l % 16.
// (a barrier that orders LDS only: loads from memory stay in flight)
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int BM, int BN> constexpr int any_result_bytes() { return BN * (BM + 4) * 4; }
template <int BM, int BN, int NT, int FM, int FN>
__device__ __forceinline__ void any_epilogue(const floatx4 (&acc)[FN][FM], const MfmaArgs &args, char *lds, int64_t m0, int64_t n0, int wm0, int wn0, int thread)
{
    constexpr int COL = (BM + 4) * 4;                  // bytes of a column (the four floats spread the sixteen columns of a block over the banks)
    const int lane = thread % 64;
    const float alpha = args.alpha, beta = args.beta;
    const int rows = static_cast<int>(args.m_main - m0 < BM ? args.m_main - m0 : BM), cols = static_cast<int>(args.n_main - n0 < BN ? args.n_main - n0 : BN);
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int i = 0; i < FM; ++i)
            *reinterpret_cast<floatx4 *>(lds + (wn0 + 16 * j + lane % 16) * COL + (wm0 + 16 * i + 4 * (lane / 16)) * 4) = acc[j][i];
    lds_barrier();
    if (args.partial != nullptr) {
        float *out = args.partial + (static_cast<int64_t>(blockIdx.z) * args.n + n0) * args.m + m0;
#pragma unroll 1
        for (int idx = thread; idx < BN * (BM / 4); idx += NT) {
            const int col = idx / (BM / 4), row = idx % (BM / 4) * 4;
            if (col >= cols) break;
            const floatx4 x = *reinterpret_cast<const floatx4 *>(lds + col * COL + row * 4);
            float *p = out + static_cast<int64_t>(col) * args.m + row;
            if (row + 4 <= rows) *reinterpret_cast<Pack<float, 4> *>(p) = Pack<float, 4>{{x.x, x.y, x.z, x.w}};
            else
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (row + e < rows) p[e] = x[e];
        }
        return;
    }
    _Float16 *out = static_cast<_Float16 *>(args.C) + n0 * args.ldc + m0;
#pragma unroll 2
    for (int idx = thread; idx < BN * (BM / 8); idx += NT) {
        const int col = idx / (BM / 8), row = idx % (BM / 8) * 8;
        if (col >= cols) break;
        _Float16 *p = out + col * args.ldc + row;
        int first = 0, last = rows - row < 8 ? rows - row : 8;         // elements first .. last - 1 of the piece are written
        const int beyond = 8 - last;
        if (args.mask != 0) {                                            // only the wanted triangle of C
            const int d = static_cast<int>(n0 - m0) + col - row;
            if (args.shape == MG_SHAPE_C_LOWER) first = d > 0 ? d : 0;
            else last = d + 1 < last ? d + 1 : last;
        }
        if (last <= first) continue;
        u32x4 old = {0u, 0u, 0u, 0u};
        // (of a piece that ends beyond the column the 16 bytes that end with it; C has eight rows or more.  Under the mask they may hold elements of the other
        // triangle, which are dropped: they lie between wanted ones in memory, and fetching the wanted ones alone, one by one, took SYRK (1161, 167) from 7.0 to 8.5 us,
        // without branches to 7.8.)
        if (beta != 0.f) old = load_unaligned_chunk<_Float16>(p - beyond);
        const floatx4 lo = *reinterpret_cast<const floatx4 *>(lds + col * COL + row * 4), hi = *reinterpret_cast<const floatx4 *>(lds + col * COL + row * 4 + 16);
        if (beyond > 0) old = shift_down(old, beyond);
        const Pack<_Float16, 8> c = __builtin_bit_cast(Pack<_Float16, 8>, old);
        Pack<_Float16, 8> o;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = alpha * (e < 4 ? lo[e % 4] : hi[e % 4]);
            o.v[e] = static_cast<_Float16>(beta != 0.f ? fmaf(beta, static_cast<float>(c.v[e]), v) : v);
        }
        if (first == 0 && last == 8) *reinterpret_cast<Pack<_Float16, 8> *>(p) = o;
        else
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (e >= first && e < last) p[e] = o.v[e];
    }
}

template <int BM, int BN, int WM, int WN, bool A_KCONTIG, bool B_KCONTIG, int DEPTH>
__global__ __launch_bounds__(WM *WN * 64) void hgemm_any_kernel(const MfmaArgs args)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using T = _Float16;
    constexpr int RB = 16, BK = 64, NT = WM * WN * 64;
    constexpr int WTM = BM / WM, WTN = BN / WN;
    constexpr int FM = WTM / RB, FN = WTN / RB;
    constexpr int KSTEPS = 2;
    static_assert(WTM % RB == 0 && WTN % RB == 0 && BM % 64 == 0 && BN % 64 == 0, "whole fragments, lines of whole 128-byte pieces");
    static_assert(DEPTH % 2 == 0, "a K-tile's LDS stage and register set go by its place in the unrolled loop");
    using LoadA = AnyLoader<BM, NT, A_KCONTIG, RB, DEPTH>;
    using LoadB = AnyLoader<BN, NT, B_KCONTIG, RB, DEPTH>;
    constexpr int A_BYTES = LoadA::LDS_BYTES, B_BYTES = LoadB::LDS_BYTES;       // LDS: [A stage 0][A stage 1][B stage 0][B stage 1]
    constexpr int SLOTS = FM * FN, FRAGS = FM + FN, PIECES = LoadA::COUNT + LoadB::COUNT;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    lds_char *const lds3 = (lds_char *)lds;

    int tm, tn;
    if (args.shape == 0) tile_coords(blockIdx.x, args.tiles_m, args.tiles_n, args.group_m, tm, tn);
    else if (BM == BN && args.shape >= MG_SHAPE_C_LOWER) tile_coords_triangle(blockIdx.x, args.tiles_m, args.shape == MG_SHAPE_C_UPPER, tm, tn);
    else tile_coords_balanced(blockIdx.x, args.tiles_m, args.tiles_n, args.group_m, args.reversed != 0, args.shape == MG_SHAPE_C_UPPER, tm, tn);
    const int64_t m0 = static_cast<int64_t>(tm) * BM, n0 = static_cast<int64_t>(tn) * BN;
    int kb = blockIdx.z * args.k_per_split;
    int ke = (kb + args.k_per_split < args.k) ? kb + args.k_per_split : args.k;
    if (!narrow_to_shape<BM, BN, BK>(args.shape, m0, n0, kb, ke)) return;

    const T *__restrict__ A = static_cast<const T *>(args.A);
    const T *__restrict__ B = static_cast<const T *>(args.B);
    const int rows_a = static_cast<int>(args.m - m0 < BM ? args.m - m0 : BM);
    const int rows_b = static_cast<int>(args.n - n0 < BN ? args.n - n0 : BN);
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int wm = wave % WM, wn = wave / WM;

    int frag_a[8], frag_b[8];          // as in hgemm_dma_tile
    auto frag_setup = [&](bool kcontig, int wrow, int operand_base, int rows, int (&frag)[8]) {
        if (kcontig) {
            const int p = operand_base + ldsmap::kcontig_base<RB>(lane, wrow);
            for (int kx = 0; kx < 4; ++kx) frag[kx] = p ^ (32 * kx);
            for (int kx = 4; kx < 8; ++kx) frag[kx] = 0;
        } else {
            for (int f = 0; f < 8; ++f) frag[f] = operand_base + ldsmap::transposed_base<RB>(lane, wrow + RB * f, rows);
        }
    };
    frag_setup(A_KCONTIG, wm * WTM, 0, BM, frag_a);
    frag_setup(B_KCONTIG, wn * WTN, 2 * A_BYTES, BN, frag_b);

    using Acc = typename BlockAcc<RB>::type;
    Acc acc[FN][FM];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int i = 0; i < FM; ++i) acc[j][i] = Acc{};

    LoadA la;
    LoadB lb;
    la.prepare(args.lda, rows_a, threadIdx.x);
    lb.prepare(args.ldb, rows_b, threadIdx.x);
    const int ktiles = (ke - kb + BK - 1) / BK;
    const int whole = (ktiles - 1) * BK, first_ks = ke - kb - whole;
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    // (a load per piece of each tile past the end costs a short sum: 128 terms took those of five K-tiles)
    auto aim_tile = [&](int t) __attribute__((always_inline)) {
        const int l0 = t == 0 ? kb + whole : (t < ktiles ? kb + (t - 1) * BK : 0);
        la.aim(A, args.lda, m0, l0, t < ktiles);
        lb.aim(B, args.ldb, n0, l0, t < ktiles);
    };
    auto load_piece = [&](auto P, auto SET) __attribute__((always_inline)) {
        constexpr int p = decltype(P)::value, set = decltype(SET)::value;
        if constexpr (p < LoadA::COUNT) la.template load<set, p>();
        else lb.template load<set, p - LoadA::COUNT>();
    };
    auto store_piece = [&](auto P, auto SET, auto PAR) __attribute__((always_inline)) {
        constexpr int p = decltype(P)::value, set = decltype(SET)::value, par = decltype(PAR)::value;
        if constexpr (p < LoadA::COUNT) la.template store<set, p>(lds + par * A_BYTES);
        else lb.template store<set, p - LoadA::COUNT>(lds + 2 * A_BYTES + par * B_BYTES);
    };
    u32x4 fa[2][FM], fb[2][FN];
    auto read_frag = [&](auto F, auto PAR, auto S, auto BUF) __attribute__((always_inline)) {
        constexpr int f = decltype(F)::value, par = decltype(PAR)::value, s = decltype(S)::value, buf = decltype(BUF)::value;
        if constexpr (f < FM) fa[buf][f] = read_tracked<A_KCONTIG, BM, f, RB, s, par * A_BYTES>(lds3, frag_a);
        else fb[buf][f - FM] = read_tracked<B_KCONTIG, BN, f - FM, RB, s, par * B_BYTES>(lds3, frag_b);
    };
    // K-tile t, the U-th of the unrolled loop, from LDS stage U % 2; tile t + 1 goes to the other stage and its registers are reloaded with tile t + 1 + DEPTH
    constexpr int TAIL = (SLOTS * MG_TAIL_SIXTEENTHS / 16) > 0 ? (SLOTS * MG_TAIL_SIXTEENTHS / 16) : 1;
    constexpr int BARRIER_SLOT = KSTEPS * SLOTS - TAIL;
    constexpr int READ_SLOTS = SLOTS >= 4 ? SLOTS * 3 / 4 : SLOTS;
    auto tile_body = [&](auto U, int t) __attribute__((always_inline)) {
        using Cur = std::integral_constant<int, decltype(U)::value % 2>;
        using Nxt = std::integral_constant<int, 1 - Cur::value>;
        using Set = std::integral_constant<int, (decltype(U)::value + 1) % DEPTH>;
        aim_tile(t + 1 + DEPTH);
        static_for<KSTEPS>([&](auto S) __attribute__((always_inline)) {
            constexpr int s = decltype(S)::value;
            static_for<SLOTS>([&](auto Q) __attribute__((always_inline)) {
                constexpr int q = decltype(Q)::value, g = s * SLOTS + q;
                if constexpr (g == BARRIER_SLOT) lds_barrier();
                mma(acc[q / FM][q % FM], fb[s & 1][q / FM], fa[s & 1][q % FM], T{});
                if constexpr (s == 0) {
                    if constexpr (q < READ_SLOTS)
                        static_for<share_begin(q + 1, FRAGS, READ_SLOTS) - share_begin(q, FRAGS, READ_SLOTS)>([&](auto R) {
                            constexpr int o = share_begin(q, FRAGS, READ_SLOTS) + decltype(R)::value;
                            read_frag(std::integral_constant<int, o < FM ? o : FM + (FRAGS - 1 - o)>{}, Cur{}, C1{}, C1{});
                        });
                } else if constexpr (g >= BARRIER_SLOT) {
                    constexpr int h = g - BARRIER_SLOT;
                    static_for<share_begin(h + 1, FRAGS, TAIL) - share_begin(h, FRAGS, TAIL)>([&](auto R) {
                        constexpr int o = share_begin(h, FRAGS, TAIL) + decltype(R)::value;
                        read_frag(std::integral_constant<int, o < FM ? o : FM + (FRAGS - 1 - o)>{}, Nxt{}, C0{}, C0{});
                    });
                }
                if constexpr (g < BARRIER_SLOT)
                    static_for<share_begin(g + 1, PIECES, BARRIER_SLOT) - share_begin(g, PIECES, BARRIER_SLOT)>([&](auto R) {
                        using P = std::integral_constant<int, share_begin(g, PIECES, BARRIER_SLOT) + decltype(R)::value>;
                        store_piece(P{}, Set{}, Nxt{});
                        load_piece(P{}, Set{});
                    });
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };

    if (ktiles > 0) {       // (a slice of a triangular operand may be empty)
        // tile 0 -> LDS stage 0, tiles 1 .. DEPTH -> registers (tile u in set u % DEPTH), first fragments
        aim_tile(0);
        static_for<LoadA::COUNT>([&](auto Q) { la.template load_end<0, decltype(Q)::value>(args.lda, rows_a, first_ks, threadIdx.x); });
        static_for<LoadB::COUNT>([&](auto Q) { lb.template load_end<0, decltype(Q)::value>(args.ldb, rows_b, first_ks, threadIdx.x); });
        static_for<DEPTH - 1>([&](auto D) {
            using Set = std::integral_constant<int, decltype(D)::value + 1>;
            aim_tile(Set::value);
            static_for<PIECES>([&](auto P) { load_piece(P, Set{}); });
        });
        static_for<LoadA::COUNT>([&](auto Q) { la.template cut<0, decltype(Q)::value>(rows_a, first_ks, threadIdx.x); });
        static_for<LoadB::COUNT>([&](auto Q) { lb.template cut<0, decltype(Q)::value>(rows_b, first_ks, threadIdx.x); });
        static_for<PIECES>([&](auto P) { store_piece(P, C0{}, C0{}); });
        aim_tile(DEPTH);
        static_for<PIECES>([&](auto P) { load_piece(P, C0{}); });
        lds_barrier();
        static_for<FRAGS>([&](auto F) { read_frag(F, C0{}, C0{}, C0{}); });
        for (int t = 0;;) {
            bool more = true;
            static_for<DEPTH>([&](auto U) __attribute__((always_inline)) {
                if (!more) return;
                tile_body(U, t);
                more = ++t < ktiles;
            });
            if (!more) break;
        }
    }
    lds_barrier();
    any_epilogue<BM, BN, NT, FM, FN>(acc, args, lds, m0, n0, wm * WTM, wn * WTN, threadIdx.x);
#else
    (void)args;
#endif
}

}  // namespace mg
