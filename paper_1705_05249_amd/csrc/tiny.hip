// GEMM for problems too small to fill the chip with macro tiles (the under-filled device of the paper's
// Section 4.6, met here by single small products rather than batches): 256^3 in FP32 is 16 tiles of 64 x 64, and
// what it costs on the macro-tile kernel is one wavefront's chain of dependent MFMAs over all of K (32 cycles per
// k: 4 us at k = 256) behind a software pipeline that needs several K-tiles to fill.
//
// Here a work-group owns one 32 x 32 block of C and its eight wavefronts share the sum: each takes an eighth of it, asks for all of its
// operands at once, turns them into MFMA operands through a part of LDS of its own (no barrier: the LDS executes a wavefront's operations in
// order), and the eight partial blocks are added through LDS by all 512 threads, which also apply alpha and beta and write C.  One
// launch, no workspace, any shape and alignment; four times as many work-groups as 64 x 64 tiles would give, each with
// an eighth of the dependent chain.
//
// Bound by latency, and for long sums by what a compute unit's L1 passes on (64 bytes a clock: 1.9 us for a block of (512, 196, 2304)).  Before,
// the work-group brought 1 KB of every row at a time into LDS, three chunks on their way and two barriers for each.  us, before / now (A along
// m and B along k): FP32 256^3 4.7 / 4.3, 512^3 7.1 / 6.2, 384 x 384 x 1024 11.3 / 8.9, (33, 65, 999) 12.1 / 8.8, 128 x 128 x 500 6.7 / 6.0; FP16 (512, 196, 2304) 10.0 / 6.9
// (both along k 8.7 / 6.2, neither 16.8 / 8.2), (256, 784, 1152) 7.0 / 5.4, 512 x 512 x 1536 8.0 / 6.2, 64 x 320 x 2560 9.9 / 6.7.
//
// Triangles: of a C of which one is wanted (SYRK) a grid of the blocks that touch it, and stores inside it only; of a triangular operand (TRMM) the
// sum from the block's first row on or up to its last.  Before, small SYRK ran on 64 x 64 tiles in slices, with a second launch.
// us, before / now: SYRK 0.81 of the time over 119 random calls, TRMM 0.91 over 99.
//
// The sum is cut into pairs of K-steps, 128 bytes of a row (64 halves, 32 floats).  MFMA blocks are 16 x 16, four to a wavefront.  A pair of an operand:
//   * along k: 32 rows of 128 bytes, eight lanes on a row: whole cache lines (16 rows of 64 bytes at a time, straight into operand registers,
//     took FP32 384 x 384 x 1024 from 10.7 to 14.3 us, both operands along k); LDS [row][k], chunk c of row r at slot c ^ swizzle16(r);
//   * FP16 along its rows: 64 lines of 64 bytes; LDS as in memory, chunk c of line k at slot c ^ 2 (k / 8 % 2), read by two transposing reads
//     per block (the 32 lanes of a pass hit 64 different banks);
//   * FP32 along its rows: four 4-byte loads per block and K-step, runs of 64 bytes, straight into the operand registers.
// Rows past the last one repeat it (they end in outputs that C does not have).  Behind the whole pairs are the values that do not fill one, with
// loads that are checked piece by piece; they include the last lines of an FP16 operand along its rows whose pieces would run past the operand's
// end (shared_sum.h), so that operands of one to three rows may leave a few values more than a pair.
#include "mfma_dma_kernel.h"
#include "mfma_host.h"
#include "shared_sum.h"

namespace mg {
namespace {

struct TinyArgs {
    const void *A, *B;
    void *C;
    int64_t a_sm, a_sk, b_sn, b_sk, ldc;     // element strides of op(A)(i, l), op(B)(l, j); one of each pair is 1
    int m, n, k;
    int share, rest;                         // work-groups per XCD, and how many XCDs have one more
    int minor, n_first;                      // blocks side by side along the shorter side of C, which is n if n_first
    int kept;                                // values of k at the end of the sum that are not in whole pairs
    int shape;                               // a triangular operand or C (enum in internal.h)
    float alpha, beta;
};

constexpr int kPairBytes = 32 * 128;                     // LDS bytes of a pair of K-steps of one operand
constexpr int kWaves = 8;

template <typename T, bool KCONTIG> struct TinySide {
    static constexpr int CH = ElemTraits<T>::CH;            // elements per 16-byte piece
    static constexpr int STEP = 4 * CH, PAIR = 2 * STEP;    // values of k per K-step and pair
    static constexpr bool HALF = sizeof(T) == 2;
    static constexpr bool TURNED = KCONTIG || HALF;         // through LDS
    static constexpr int PIECES = 4;                        // 16-byte pieces of a pair per lane

    // Addresses are a wave-uniform part (64 bits, scalar) and a lane's byte offset that is the same for every pair.
    const char *base;           // the block's first row at pair 0 of this wavefront
    int64_t ld;                 // bytes
    int rows_left;              // rows of the operand behind the block's first one
    int row, k;                 // of this lane's first piece or element: row of the block and value of k inside the pair
    uint32_t at[KCONTIG ? PIECES : (HALF ? 1 : 2)];

    // lane's piece i of a pair: along k, row lane / 8 + 8 i, chunk lane % 8; else line lane / 4 + 16 i, chunk lane % 4
    __device__ inline void prepare(const void *data, int64_t ld_, int rows, int row0, int64_t k0, int lane)
    {
        ld = ld_ * static_cast<int64_t>(sizeof(T));
        rows_left = rows - 1 - row0;
        base = static_cast<const char *>(data) + (KCONTIG ? row0 * ld + k0 * static_cast<int64_t>(sizeof(T)) : row0 * static_cast<int64_t>(sizeof(T)) + k0 * ld);
        if constexpr (KCONTIG) {
            row = lane / 8;
            k = lane % 8 * CH;
#pragma unroll
            for (int i = 0; i < PIECES; ++i) at[i] = static_cast<uint32_t>(existing(row + 8 * i) * ld + k * static_cast<int>(sizeof(T)));
        } else if constexpr (HALF) {
            row = lane % 4 * CH;
            row = row <= rows_left ? row : 0;          // (a piece without rows: the first one again)
            k = lane / 4;
            at[0] = static_cast<uint32_t>(row * 2 + k * ld);
        } else {
            row = lane % 16;
            k = lane / 16 * 4;
#pragma unroll
            for (int b = 0; b < 2; ++b) at[b] = static_cast<uint32_t>(existing(row + 16 * b) * 4 + k * ld);
        }
    }
    __device__ inline int existing(int r) const { return r < rows_left ? r : rows_left; }

    // wave-uniform address of pair number `pair` of this wavefront, `l` values of k on
    __device__ inline const char *line(int pair, int l) const
    {
        const int64_t from = static_cast<int64_t>(pair) * PAIR + l;
        return base + (KCONTIG ? from * static_cast<int64_t>(sizeof(T)) : from * ld);
    }
    __device__ static inline const T *element(const char *uniform, uint32_t lane_offset) { return reinterpret_cast<const T *>(uniform + lane_offset); }

    // FP32 along its rows: the pairs from `pair` on by buffer loads, whose scalar offsets take the place of 64-bit addresses in vector registers
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ inline void aim(int pair)
    {
        if constexpr (!TURNED) rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(line(pair, 0)), 0, 0x7fffffff, 0x00020000);
    }

    // pair number `pair` of this wavefront, the J-th behind the one aimed at
    template <int J> __device__ inline void fetch(u32x4 (&f)[PIECES], int pair) const
    {
        if constexpr (KCONTIG) {
#pragma unroll
            for (int i = 0; i < PIECES; ++i) f[i] = load_unaligned_chunk<T>(element(line(pair, 0), at[i]));
        } else if constexpr (HALF) {
#pragma unroll
            for (int i = 0; i < PIECES; ++i) f[i] = load_unaligned_chunk<T>(element(line(pair, 16 * i), at[0]));
        } else {
            // operand 2 s + b: K-step s, block b
#pragma unroll
            for (int i = 0; i < PIECES; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    f[i][e] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, at[i % 2], static_cast<uint32_t>(ld) * (J * PAIR + i / 2 * STEP + e), 0);
        }
    }

    // pair number `pair` of this wavefront, of which `left` values of k exist (or all)
    __device__ inline void fetch_rest(u32x4 (&f)[PIECES], int pair, int left) const
    {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if constexpr (KCONTIG) {
                const T *p = element(line(pair, 0), at[i]);
                if (left - k >= CH) v = load_unaligned_chunk<T>(p);
                else if (left - k > 0) v = gather_chunk<T>(p, left - k);
            } else if constexpr (HALF) {
                const T *p = element(line(pair, 16 * i), at[0]);
                const int valid = rows_left + 1 - row;
                if (k + 16 * i < left) v = valid >= CH ? load_unaligned_chunk<T>(p) : gather_chunk<T>(p, valid);
            } else {
                // (a descriptor that ends with the last line: what lies behind it reads as zero, without a branch for each element; the whole
                // offset is the lane's, the scalar one is no part of the check; with branches 128 x 128 x 500 took 6.7 us instead of 6.0, 136 x 151 x 136
                // 4.8 instead of 4.3)
                const __amdgpu_buffer_rsrc_t rest = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(line(pair, 0)), 0, static_cast<int>(ld) * left, 0x00020000);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_raw_buffer_load_b32(rest, at[i % 2] + static_cast<uint32_t>(ld) * (i / 2 * STEP + e), 0, 0);
            }
            f[i] = v;
        }
    }

    // pieces -> operands: f[2 s + b] becomes K-step s of block b
    __device__ inline void turn(u32x4 (&f)[PIECES], lds_char *mine, int lane) const
    {
        if constexpr (TURNED) {
            using lds_u32x4 = __attribute__((address_space(3))) u32x4;
            const int ln = lane % 16, lg = lane / 16;
#pragma unroll
            for (int i = 0; i < PIECES; ++i) {
                const int to = KCONTIG ? ldsmap::kcontig_slot<16>(lane / 8 + 8 * i, lane % 8)
                                       : (lane / 4 + 16 * i) * 64 + (((lane % 4) ^ (2 * (((lane / 4) >> 3) & 1))) << 4);
                *(lds_u32x4 *)(mine + to) = f[i];
            }
#pragma unroll
            for (int i = 0; i < PIECES; ++i) {
                const int s = i / 2, b = i % 2;
                if constexpr (KCONTIG) {
                    f[i] = *(lds_u32x4 *)(mine + ldsmap::kcontig_slot<16>(16 * b + ln, 4 * s + lg));
                } else {
                    const int quad = ln % 4, line = 32 * s + 8 * lg + ln / 4;
                    lds_char *const p = mine + line * 64 + (((2 * b + quad / 2) ^ (2 * (lg & 1))) << 4) + 8 * (quad % 2);
                    const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)p);
                    const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)(p + 4 * 64));
                    f[i] = __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
            }
        }
    }
};

// SHAPED: with a triangular operand or C (the tests of the shape cost the others 0.1 us: 256^3 4.36 / 4.47)
template <typename T, bool A_KCONTIG, bool B_KCONTIG, bool SHAPED>
__global__ __launch_bounds__(kWaves * 64) void tiny_gemm_kernel(const TinyArgs a)
{
#if defined(__HIP_DEVICE_COMPILE__)      // the host pass needs the kernel's symbol only (LDS address-space code is device code)
    using SideA = TinySide<T, A_KCONTIG>;
    using SideB = TinySide<T, B_KCONTIG>;
    constexpr int PAIR = SideA::PAIR;
    constexpr int NP = sizeof(T) == 4 ? 4 : 5;          // pairs whose loads are in flight together: FP32 sums up to 1024, FP16 up to 2560
    extern __shared__ __attribute__((aligned(16))) char lds[];

    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    // Blocks of one XCD (ids 8 apart) lie side by side, along the shorter side of C first: its L2 then fetches an eighth of the
    // larger operand instead of all of it.  Before / after, us: (150, 1500, 600) FP32 11.8 / 9.7, FP16 (512, 196, 2304) 10.9 / 9.9,
    // (300, 800, 1500) 12.3 / 10.2, (190, 1200, 2000) 10.5 / 8.9.
    int m0, n0;
    if (!SHAPED || a.shape < MG_SHAPE_C_LOWER) {
        const int xcd = blockIdx.x % 8;
        const int id = xcd * a.share + (xcd < a.rest ? xcd : a.rest) + blockIdx.x / 8;
        const int outer = id / a.minor, inner = id - outer * a.minor;
        m0 = (a.n_first ? outer : inner) * 32;
        n0 = (a.n_first ? inner : outer) * 32;
    } else {                                           // a work-group for each block that touches the wanted triangle
        tile_coords_triangle(blockIdx.x, a.minor, a.shape == MG_SHAPE_C_UPPER, m0, n0);
        m0 *= 32;
        n0 *= 32;
    }
    int kb = 0, ke = a.k;
    if constexpr (SHAPED) narrow_to_shape<32, 32, 32>(a.shape, m0, n0, kb, ke);

    // whole pairs, an eighth to each wavefront; what is left is the last wavefront's
    const int pairs = whole_pairs(ke - kb, a.kept, PAIR), share = (pairs + kWaves - 1) / kWaves;
    const int begin = wave * share < pairs ? wave * share : pairs, count = begin + share < pairs ? share : pairs - begin;
    const int left = wave == kWaves - 1 ? ke - kb - pairs * PAIR : 0;
    SideA sa;
    SideB sb;
    sa.prepare(a.A, A_KCONTIG ? a.a_sm : a.a_sk, a.m, m0, kb + static_cast<int64_t>(begin) * PAIR, lane);
    sb.prepare(a.B, B_KCONTIG ? a.b_sn : a.b_sk, a.n, n0, kb + static_cast<int64_t>(begin) * PAIR, lane);
    lds_char *const mine_a = (lds_char *)lds + wave * (SideA::TURNED + SideB::TURNED) * kPairBytes;
    lds_char *const mine_b = mine_a + SideA::TURNED * kPairBytes;

    // this thread's two elements of C (row tid % 32, columns tid / 32 and + 16): the old values are asked for now
    T *C = static_cast<T *>(a.C);
    bool mine[2];
    float old[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int mi = tid % 32, ni = tid / 32 + 16 * i;
        mine[i] = m0 + mi < a.m && n0 + ni < a.n;
        if (SHAPED && a.shape == MG_SHAPE_C_LOWER) mine[i] = mine[i] && m0 + mi >= n0 + ni;
        if (SHAPED && a.shape == MG_SHAPE_C_UPPER) mine[i] = mine[i] && m0 + mi <= n0 + ni;
        if (mine[i] && a.beta != 0.f) old[i] = load_as_float(C + (m0 + mi) + (n0 + ni) * a.ldc);
    }
    // [n][m]; FP32: four sets, by value of k modulo 4 of a lane's piece, added pairwise at the end.  A wavefront's share is whole pairs, so with one
    // set a short sum would be chains of 32 terms on few wavefronts, and its error against 64 bits 1.4 times that of an eighth for each (k = 64).
    constexpr int SETS = sizeof(T) == 4 ? 4 : 1;
    floatx4 acc[SETS][2][2] = {};
    auto multiply = [&](u32x4 (&x)[4], u32x4 (&y)[4]) __attribute__((always_inline)) {
        sa.turn(x, mine_a, lane);
        sb.turn(y, mine_b, lane);
        static_for<2>([&](auto S) __attribute__((always_inline)) {
            constexpr int s = 2 * decltype(S)::value;
            if constexpr (sizeof(T) == 2) {
                mma(acc[0][0][0], y[s], x[s], T{});
                mma(acc[0][0][1], y[s], x[s + 1], T{});
                mma(acc[0][1][0], y[s + 1], x[s], T{});
                mma(acc[0][1][1], y[s + 1], x[s + 1], T{});
            } else {
                // (whole-vector casts and named components, see mma; the four blocks in turn: an instruction does not wait for the one before)
                const floatx4 u0 = __builtin_bit_cast(floatx4, x[s]), u1 = __builtin_bit_cast(floatx4, x[s + 1]);
                const floatx4 v0 = __builtin_bit_cast(floatx4, y[s]), v1 = __builtin_bit_cast(floatx4, y[s + 1]);
                auto blocks = [&](floatx4 (&c)[2][2], float p, float q, float r, float t) __attribute__((always_inline)) {
                    c[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(p, r, c[0][0], 0, 0, 0);
                    c[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(q, r, c[0][1], 0, 0, 0);
                    c[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(p, t, c[1][0], 0, 0, 0);
                    c[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(q, t, c[1][1], 0, 0, 0);
                };
                blocks(acc[0], u0.x, u1.x, v0.x, v1.x);
                blocks(acc[1], u0.y, u1.y, v0.y, v1.y);
                blocks(acc[2], u0.z, u1.z, v0.z, v1.z);
                blocks(acc[3], u0.w, u1.w, v0.w, v1.w);
            }
        });
    };
    for (int done = 0; done < count; done += NP) {
        u32x4 fa[NP][4], fb[NP][4];
        sa.aim(done);
        sb.aim(done);
        static_for<NP>([&](auto J) __attribute__((always_inline)) {
            constexpr int j = decltype(J)::value;
            if (done + j < count) {
                sa.template fetch<j>(fa[j], done + j);
                sb.template fetch<j>(fb[j], done + j);
            }
        });
        asm volatile("" ::: "memory");             // all loads first: merged with the products they would wait for each other
        static_for<NP>([&](auto J) __attribute__((always_inline)) {
            constexpr int j = decltype(J)::value;
            if (done + j < count) multiply(fa[j], fb[j]);
        });
    }
    // (twice only for an FP16 operand of one to three rows)
    for (int rest = left, pair = count; rest > 0; rest -= PAIR, ++pair) {
        u32x4 x[4], y[4];
        sa.fetch_rest(x, pair, rest);
        sb.fetch_rest(y, pair, rest);
        multiply(x, y);
    }
    if constexpr (SETS == 4) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[0][j][i] = (acc[0][j][i] + acc[1][j][i]) + (acc[2][j][i] + acc[3][j][i]);
    }
    // The eight partial blocks -> LDS as [wavefront][register][lane] (register 8 j + 4 i + r of lane l is
    // C(16 i + 4 (l / 16) + r, 16 j + l % 16)); every thread adds the eight values of two (register, lane) pairs, hands the
    // sums on through a [column][row] staging area (33 floats per column: no bank conflicts either way), and writes
    // two elements of C, consecutive threads consecutive rows.
    __syncthreads();
    float *part = reinterpret_cast<float *>(lds);
    float *stage = reinterpret_cast<float *>(lds + kWaves * 16 * 64 * 4);
#pragma unroll
    for (int r = 0; r < 16; ++r) part[(wave * 16 + r) * 64 + lane] = acc[0][r / 8][r / 4 % 2][r % 4];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = tid + 512 * i, r = e / 64, l = e % 64;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += part[w * 1024 + e];
        stage[(16 * (r / 8) + l % 16) * 33 + 16 * (r / 4 % 2) + 4 * (l / 16) + r % 4] = sum;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int mi = tid % 32, ni = tid / 32 + 16 * i;
        if (mine[i]) {
            float o = a.alpha * stage[ni * 33 + mi];
            if (a.beta != 0.f) o = fmaf(a.beta, old[i], o);
            store_from_float(C + (m0 + mi) + (n0 + ni) * a.ldc, o);
        }
    }
#else
    (void)a;
#endif
}

template <typename T, bool AK, bool BKC> struct TinyConfig {
    static constexpr int DTYPE = sizeof(T) == 4 ? MG_F32 : MG_F16;
    static constexpr int SUMS = kWaves * 16 * 64 * 4 + 32 * 33 * 4;
    static constexpr int PAIRS = kWaves * (TinySide<T, AK>::TURNED + TinySide<T, BKC>::TURNED) * kPairBytes;
    static constexpr int LDS = PAIRS > SUMS ? PAIRS : SUMS;

    static bool legal(const Problem &p, int split, int64_t alignment)
    {
        (void)alignment;
        if (p.dtype != DTYPE || p.a_trans != AK || p.b_trans == BKC || split != 1) return false;
        if (p.conv != nullptr || p.fringe_m != 0 || p.fringe_n != 0 || p.clip_m != 0 || p.clip_n != 0) return false;
        if (p.alpha == 0.f || p.k == 0 || (p.shape >= MG_SHAPE_C_LOWER && p.m != p.n)) return false;
        if (p.m >= (int64_t(1) << 31) || p.n >= (int64_t(1) << 31) || p.k >= (int64_t(1) << 31)) return false;
        // (offsets inside the pairs of K-steps that are loaded together)
        if ((p.lda > p.ldb ? p.lda : p.ldb) * 192 * static_cast<int64_t>(sizeof(T)) >= (int64_t(1) << 31)) return false;
        return ceil_div(p.m, 32) * ceil_div(p.n, 32) < (int64_t(1) << 31);
    }

    static size_t workspace(const Problem &, int) { return 0; }

    static hipError_t launch(const Problem &p, int) { return p.shape == MG_SHAPE_GENERAL ? launch_flavour<false>(p) : launch_flavour<true>(p); }

    template <bool SHAPED> static hipError_t launch_flavour(const Problem &p)
    {
        static bool attr_set = false;
        auto kernel = tiny_gemm_kernel<T, AK, BKC, SHAPED>;
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        TinyArgs a{};
        a.A = p.A; a.B = p.B; a.C = p.C;
        a.a_sm = p.a_sm(); a.a_sk = p.a_sk(); a.b_sn = p.b_sn(); a.b_sk = p.b_sk(); a.ldc = p.ldc;
        a.m = static_cast<int>(p.m); a.n = static_cast<int>(p.n); a.k = static_cast<int>(p.k);
        a.alpha = p.alpha; a.beta = p.beta;
        const int64_t blocks_m = ceil_div(p.m, 32);
        const unsigned groups = static_cast<unsigned>(p.shape >= MG_SHAPE_C_LOWER ? blocks_m * (blocks_m + 1) / 2 : blocks_m * ceil_div(p.n, 32));
        a.share = static_cast<int>(groups / 8);
        a.rest = static_cast<int>(groups % 8);
        a.n_first = p.m >= p.n ? 1 : 0;
        a.minor = static_cast<int>(ceil_div(a.n_first ? p.n : p.m, 32));
        a.shape = p.shape;
        const int piece = sizeof(T) == 2 ? 8 : 1;            // (FP32 operands along their rows come in single elements)
        const int kept_a = AK ? 0 : lines_kept_back(p.m, p.lda, piece), kept_b = BKC ? 0 : lines_kept_back(p.n, p.ldb, piece);
        a.kept = kept_a > kept_b ? kept_a : kept_b;
        hipLaunchKernelGGL(kernel, dim3(groups), dim3(512), LDS, p.stream, a);
        return hipGetLastError();
    }

    static KernelEntry entry(const char *name)
    {
        mg_config c{};
        c.family = MG_FAMILY_MFMA;
        c.dtype = DTYPE;
        c.tile_m = 32; c.tile_n = 32; c.tile_k = TinySide<T, AK>::PAIR;
        c.waves_m = 1; c.waves_n = 1;
        c.split_k = 1;
        c.threads = 512;
        c.lds_bytes = LDS;
        KernelEntry e{name, c, legal, workspace, launch, nullptr, nullptr};
        e.masks_triangle = true;
        return e;
    }
};

}  // namespace

// Names: <t>tiny_32x32_<a><b>, a/b = k or m/n: which direction the operand is contiguous in.
void register_tiny(std::vector<KernelEntry> &table)
{
    table.push_back(TinyConfig<float, false, true>::entry("stiny_32x32_mk"));
    table.push_back(TinyConfig<float, true, true>::entry("stiny_32x32_kk"));
    table.push_back(TinyConfig<float, false, false>::entry("stiny_32x32_mn"));
    table.push_back(TinyConfig<float, true, false>::entry("stiny_32x32_kn"));
    table.push_back(TinyConfig<_Float16, false, true>::entry("htiny_32x32_mk"));
    table.push_back(TinyConfig<_Float16, true, true>::entry("htiny_32x32_kk"));
    table.push_back(TinyConfig<_Float16, false, false>::entry("htiny_32x32_mn"));
    table.push_back(TinyConfig<_Float16, true, false>::entry("htiny_32x32_kn"));
}

}  // namespace mg
