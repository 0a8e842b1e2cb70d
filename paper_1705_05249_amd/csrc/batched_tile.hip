// Batched GEMM for instances of any shape (paper Section 4.6): one tile of one instance per team of wavefronts, operands
// staged through LDS, MFMA 16x16 blocks; FP32, and FP16 storage with FP32 accumulation.
//
// What bounds a batched call is memory: an instance is read and written once and its sum is at most a few hundred
// terms.  So the kernel is built around how it asks for memory, not around the MFMA pipeline:
//   * operands are fetched line by line (a line: the contiguous direction, a row of op(A) along k or a k line along m) in
//     16-byte pieces at element alignment, consecutive lanes on consecutive pieces, whatever the extents and leading
//     dimensions are; a line's last piece may run into the next line (those elements are zeroed, or belong to rows that
//     are never stored), only the last piece of the matrix itself is gathered element by element;
//   * the pieces of the next chunk of k are on their way while the MFMAs of the current one run, and several teams
//     share a compute unit (12 to 20 KB of LDS each; the four one-wavefront teams of a work-group 32 to 48), so loads of some overlap the arithmetic of others;
//   * results go through LDS, 16 columns per wavefront column at a time, and leave as 16-byte pieces along the columns of C.
// LDS layouts: an operand along k as [row][k] in 128-byte rows with swizzled chunks (lds_layout.h, 16-row fragments); an
// operand along m / n as it lies in memory, [k][row], lines padded by 16 (FP32) or 32 bytes (FP16) so that the 16 or 32 lanes
// that the LDS serves at once hit different banks.  FP16 fragments of the latter are transposing reads.
// A K-step is 16 values of k: lane (r = lane % 16, g = lane / 16) holds X[r][4g + s], s = 0..3, the operand of one
// v_mfma_f32_16x16x16_f16, or of four v_mfma_f32_16x16x4_f32.  (The 16x16x32 form would halve the MFMA time, which is a fifth
// of the memory time, and cost the [k][row] layout its conflict-free reads.)
// Measured (us; the FMA kernel or the register-resident 64-wide blocks these instances ran on before / this): 512 x (128, 128, 64)
// FP16 40.0 / 9.9 (33 MB, 3.4 TB/s, the launch included), FP32 30.6 / 19.8; FP16 64^3 (3111, both transposed) 46 / 17.5, 81^3 (800)
// 105 / 15, (19, 80, 144) x 2100 171 / 23; FP32 64^3 (5000, B along n) 103 / 69 (328 MB, 4.8 TB/s), 93^3 (856) 63 / 31, 99^3 (4122)
// 313 / 191: there the MFMAs of the padded blocks take half of the time and do not hide behind the loads.
// The piece that a column of C ends in takes its old values from the 16 bytes that end with the column and goes out as 8, 4 and 2 bytes; element by
// element, each behind its old value, it cost a memory latency per element (FP32 73^3, 569 instances, beta 22.2 / 19.4; FP16 121 x 150 x 27 62 / 42).
// A team skips the columns of 16x16 blocks that the instance does not have, and its columns of blocks are dealt out evenly.
#include "batched_walk.h"
#include "mfma_any_kernel.h"

namespace mg {
namespace {

typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));

struct TileBatchArgs {
    const void *A, *B;
    void *C;
    const int64_t *a_off, *b_off, *c_off;
    const float *alphas, *betas;
    int64_t lda, ldb, ldc;
    int m, n, k;
    batchwalk::Divisor tiles_m;    // tiles along m
    int64_t batch;                 // of this launch: the instances behind the pointers and offsets,
    uint32_t tile0;                // and the tiles of each from tile0 on
    batchwalk::Walk walk;
    int strided;
    int64_t stride_a, stride_b, stride_c;
    float alpha, beta;
};

// idx / d for idx < 4096, d <= 64 (ceil(2^20 / d) is exact there)
struct SmallDiv {
    uint32_t d, magic;
    __device__ explicit SmallDiv(int by) : d(by), magic((((1u << 20) + by - 1) / by)) {}
    __device__ inline int quot(int idx) const { return static_cast<int>((static_cast<uint32_t>(idx) * magic) >> 20); }
};

// One operand of a tile: memory -> registers -> LDS.  ROWS: rows of the tile; NT: threads of the team.
template <typename T, int ROWS, int NT, bool KCONTIG> struct PanelLoader {
    static constexpr int V = ElemTraits<T>::CH;                      // elements per piece
    static constexpr int KC = 128 / static_cast<int>(sizeof(T));     // values of k per chunk
    static constexpr int PAD = sizeof(T) == 4 ? 16 : 32;
    static constexpr int LINE = ROWS * static_cast<int>(sizeof(T)) + PAD;      // [k][row] layout: bytes per line
    static constexpr int BYTES = KCONTIG ? ROWS * 128 : KC * LINE;
    static constexpr int U = ROWS * 8 / NT;                          // pieces per thread
    static_assert(U * NT == ROWS * 8, "whole pieces per thread");
    u32x4 regs[U];
    const T *at[U];            // where piece i of this thread lies in the chunk to come
    int line[U], place[U];     // its line and its first element's place in the line (elements)
    int64_t step;              // elements from a chunk to the next

    // X: first element of the tile.  Pieces are numbered along the lines: eight per row of k values, or as many as the
    // tile's rows take.
    __device__ inline void prepare(const T *X, int64_t ld, int rows, int tid)
    {
        const SmallDiv per_line((rows + V - 1) / V);
        static_for<U>([&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            const int idx = tid + i * NT;
            line[i] = KCONTIG ? idx / 8 : per_line.quot(idx);
            place[i] = (KCONTIG ? idx % 8 : idx - line[i] * static_cast<int>(per_line.d)) * V;
            at[i] = X + line[i] * ld + place[i];
        });
        step = KCONTIG ? KC : KC * ld;
    }

    // The next chunk, kleft values of k before the end of the sum; rows of the tile, rows_end: rows of the matrix from the tile's
    // first row on.
    __device__ inline void load(int64_t ld, int rows, int rows_end, int kleft)
    {
        static_for<U>([&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            u32x4 v = {0u, 0u, 0u, 0u};
            const int valid = (KCONTIG ? kleft : rows) - place[i];
            if ((KCONTIG ? line[i] < rows : line[i] < kleft && line[i] < KC) && valid > 0) {
                // elements past the end of a line are in bounds while enough of the matrix follows
                const int behind = (KCONTIG ? rows_end : kleft) - 1 - line[i];
                if (valid >= V || (behind < V ? behind : V) * ld >= V) v = load_unaligned_chunk<T>(at[i]);
                else v = gather_chunk<T>(at[i], valid);
            }
            regs[i] = v;
            at[i] += step;
        });
    }

    __device__ inline void store(char *lds, int rows, int kleft)
    {
        static_for<U>([&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            if constexpr (KCONTIG) {                     // values of k past the end count as zero
                const int valid = kleft - place[i];
                if (valid < V)
                    static_for<4>([&](auto D) {
                        constexpr int d = decltype(D)::value;
                        if constexpr (sizeof(T) == 4) regs[i][d] = d < valid ? regs[i][d] : 0u;
                        else regs[i][d] = 2 * d + 1 < valid ? regs[i][d] : (2 * d < valid ? regs[i][d] & 0xffffu : 0u);
                    });
            }
            if (line[i] < (KCONTIG ? rows : KC))
                *reinterpret_cast<u32x4 *>(lds + (KCONTIG ? ldsmap::kcontig_slot<16>(line[i], place[i] / V)
                                                          : line[i] * LINE + place[i] * static_cast<int>(sizeof(T)))) = regs[i];
        });
    }
};

// Lane's fragment of rows row0 .. row0 + 15 at K-step s
template <bool KCONTIG, int LINE> __device__ inline floatx4 read_fragment(char *lds, int row0, int s, int lane, float)
{
    const int r = lane % 16, g = lane / 16;
    if constexpr (KCONTIG) {
        return *reinterpret_cast<const floatx4 *>(lds + ldsmap::kcontig_slot<16>(row0 + r, 4 * s + g));
    } else {
        const char *p = lds + (16 * s + 4 * g) * LINE + (row0 + r) * 4;
        return floatx4{*reinterpret_cast<const float *>(p), *reinterpret_cast<const float *>(p + LINE),
                       *reinterpret_cast<const float *>(p + 2 * LINE), *reinterpret_cast<const float *>(p + 3 * LINE)};
    }
}
template <bool KCONTIG, int LINE> __device__ inline halfx4 read_fragment(char *lds, int row0, int s, int lane, _Float16)
{
    const int r = lane % 16, g = lane / 16;
    if constexpr (KCONTIG) {
        return *reinterpret_cast<const halfx4 *>(lds + ldsmap::kcontig_slot<16>(row0 + r, 2 * s + g / 2) + 8 * (g & 1));
    } else {
#if defined(__HIP_DEVICE_COMPILE__)
        // (lane r of a group of 16 fetches four rows at one line, and receives four lines of row r: see lds_layout.h)
        typedef short shortx4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) shortx4 lds_shortx4;
        char *p = lds + (16 * s + 4 * g + r / 4) * LINE + (row0 + 4 * (r % 4)) * 2;
        return __builtin_bit_cast(halfx4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)p));
#else
        return halfx4{};
#endif
    }
}

// one K-step of the first N blocks of a column of blocks, no MFMA waiting for the one before it
template <int N, int MB> __device__ inline void step_mma(const floatx4 (&x)[N], floatx4 y, floatx4 (&c)[MB])
{
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < N; ++i) c[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i][e], y[e], c[i], 0, 0, 0);
}
template <int N, int MB> __device__ inline void step_mma(const halfx4 (&x)[N], halfx4 y, floatx4 (&c)[MB])
{
#pragma unroll
    for (int i = 0; i < N; ++i) c[i] = __builtin_amdgcn_mfma_f32_16x16x16f16(x[i], y, c[i], 0, 0, 0);
}

// LDS of a work-group: the operands' chunks of each team, or two strips of its results (floats, columns padded by four)
template <typename T, int WM, int WN, int MB, int NB, bool A_KC, bool B_KC> struct TileLds {
    static constexpr int TEAM = WM * WN, TM = WM * MB * 16, TN = WN * NB * 16;
    static constexpr int OPERANDS = PanelLoader<T, TM, TEAM * 64, A_KC>::BYTES + PanelLoader<T, TN, TEAM * 64, B_KC>::BYTES;
    static constexpr int STAGE_LD = TM + 4, STAGE = WN * 16 * STAGE_LD * 4;
    static constexpr int PER_TEAM = OPERANDS > 2 * STAGE ? OPERANDS : 2 * STAGE;
    static constexpr int BYTES = 4 / TEAM * PER_TEAM;
};

// WM x WN wavefronts make a team; each owns up to MB x NB blocks of 16 x 16.  A work-group is four wavefronts: one team of
// four, or four teams of one (instances of at most 32 x 32; no barrier anywhere then).
template <typename T, int WM, int WN, int MB, int NB, bool A_KC, bool B_KC>
__global__ __launch_bounds__(256) void batched_tile_kernel(const TileBatchArgs a)
{
    constexpr int TEAM = WM * WN, NT = TEAM * 64, TM = WM * MB * 16, TN = WN * NB * 16;
    static_assert(TEAM == 1 || TEAM == 4, "a team is a wavefront or a work-group");
    using LoadA = PanelLoader<T, TM, NT, A_KC>;
    using LoadB = PanelLoader<T, TN, NT, B_KC>;
    constexpr int KC = LoadA::KC;
    using Lds = TileLds<T, WM, WN, MB, NB, A_KC, B_KC>;
    constexpr int STAGE_LD = Lds::STAGE_LD, STAGE = Lds::STAGE;
    __shared__ __attribute__((aligned(16))) char shared[Lds::BYTES];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int tid = TEAM == 1 ? lane : static_cast<int>(threadIdx.x);
    char *lds = shared + (TEAM == 1 ? wave * Lds::PER_TEAM : 0);
    auto meet = [] {
        if constexpr (TEAM == 1) {
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    };

    int64_t inst;
    uint32_t tile = 0;
    if constexpr (TEAM == 1) {
        inst = static_cast<int64_t>(blockIdx.x) * 4 + wave;
    } else {
        const batchwalk::Place at = batchwalk::place(a.walk, blockIdx.x);
        inst = at.inst;
        tile = a.tile0 + at.tile;
    }
    if (inst >= a.batch) return;
    const float alpha = a.strided ? a.alpha : a.alphas[inst], beta = a.strided ? a.beta : a.betas[inst];
    const uint32_t tile_col = a.tiles_m.quot(tile);
    const int i0 = static_cast<int>(tile - tile_col * a.tiles_m.d) * TM, j0 = static_cast<int>(tile_col) * TN;
    const int mt = a.m - i0 < TM ? a.m - i0 : TM, nt = a.n - j0 < TN ? a.n - j0 : TN;
    const T *A = static_cast<const T *>(a.A) + (a.strided ? inst * a.stride_a : a.a_off[inst]) + (A_KC ? i0 * a.lda : i0);
    const T *B = static_cast<const T *>(a.B) + (a.strided ? inst * a.stride_b : a.b_off[inst]) + (B_KC ? j0 * a.ldb : j0);
    T *C = static_cast<T *>(a.C) + (a.strided ? inst * a.stride_c : a.c_off[inst]) + i0 + j0 * a.ldc;
    const int k = alpha == 0.f ? 0 : a.k;                              // alpha == 0: A and B are not read at all

    // Columns of blocks are dealt out evenly, the last wavefront column getting what is left; which wavefront (and so which
    // SIMD) that is changes from work-group to work-group.  Rows of blocks are a compile-time matter (the tile is chosen to fit).
    const int role = TEAM == 1 ? 0 : (wave + static_cast<int>(blockIdx.x / 8)) & 3;
    const int wm = role % WM, wn = role / WM;
    const int blocks_n = (nt + 15) / 16, nb_even = (blocks_n + WN - 1) / WN;
    const int row0 = wm * MB * 16, col0 = wn * nb_even * 16;
    const int nb = min(nb_even, blocks_n - wn * nb_even);

    floatx4 acc[NB][MB];
#pragma unroll
    for (int bj = 0; bj < NB; ++bj)
#pragma unroll
        for (int bi = 0; bi < MB; ++bi) acc[bj][bi] = floatx4{0.f, 0.f, 0.f, 0.f};

    // Results leave in strips: strip bj is column block bj of every wavefront column, [16 WN columns][rows] floats in LDS.
    // A thread's pieces of a strip (PER consecutive rows of one column):
    constexpr int PER = ElemTraits<T>::CH;
    constexpr int PASSES = (WN * 16 * (TM / PER) + NT - 1) / NT;
    const SmallDiv per_col((mt + PER - 1) / PER);
    int piece_c[PASSES], piece_row[PASSES];
    static_for<PASSES>([&](auto P) {
        constexpr int p = decltype(P)::value;
        const int idx = tid + p * NT;
        piece_c[p] = per_col.quot(idx);
        piece_row[p] = (idx - piece_c[p] * static_cast<int>(per_col.d)) * PER;
    });
    auto column = [&](int c, int bj) { return (c / 16 * nb_even + bj) * 16 + c % 16; };
    auto has = [&](int c, int bj) { return c < WN * 16 && bj < nb_even && column(c, bj) < nt; };
    // old values of the strip after the one that is being written
    Pack<T, PER> old[PASSES];
    auto fetch_old = [&](int bj) __attribute__((always_inline)) {
        if (beta == 0.f) return;
        static_for<PASSES>([&](auto P) __attribute__((always_inline)) {
            constexpr int p = decltype(P)::value;
            // (of a piece that ends beyond the column the 16 bytes that end with it)
            const int beyond = piece_row[p] + PER > mt ? piece_row[p] + PER - mt : 0;
            if (has(piece_c[p], bj) && a.m >= PER)
                old[p] = *reinterpret_cast<const Pack<T, PER> *>(C + column(piece_c[p], bj) * a.ldc + piece_row[p] - beyond);
        });
    };

    LoadA la;
    LoadB lb;
    if (k > 0) {
        la.prepare(A, a.lda, mt, tid);
        lb.prepare(B, a.ldb, nt, tid);
        la.load(a.lda, mt, a.m - i0, k);
        lb.load(a.ldb, nt, a.n - j0, k);
    }
    fetch_old(0);
    batchwalk::for_chunks<KC>(k, [&](int left) __attribute__((always_inline)) {
        if (left < k) meet();                                          // everyone is done with the chunk before
        la.store(lds, mt, left);
        lb.store(lds + LoadA::BYTES, nt, left);
        meet();
        if (left > KC) {
            la.load(a.lda, mt, a.m - i0, left - KC);
            lb.load(a.ldb, nt, a.n - j0, left - KC);
        }
        static_for<KC / 16>([&](auto S) __attribute__((always_inline)) {
            constexpr int s = decltype(S)::value;
            if (left <= s * 16) return;
            using Frag = decltype(read_fragment<A_KC, LoadA::LINE>(lds, 0, 0, 0, T{}));
            Frag fa[MB], fb[NB];
#pragma unroll
            for (int bi = 0; bi < MB; ++bi) fa[bi] = read_fragment<A_KC, LoadA::LINE>(lds, row0 + bi * 16, s, lane, T{});
#pragma unroll
            for (int bj = 0; bj < NB; ++bj) fb[bj] = read_fragment<B_KC, LoadB::LINE>(lds + LoadA::BYTES, col0 + bj * 16, s, lane, T{});
#pragma unroll
            for (int bj = 0; bj < NB; ++bj)
                if (bj < nb) step_mma(fa, fb[bj], acc[bj]);
        });
    });

    meet();
    static_for<NB>([&](auto J) __attribute__((always_inline)) {
        constexpr int bj = decltype(J)::value;
        if (bj >= nb_even) return;
        char *stage = lds + (bj & 1) * STAGE;                          // two strips in turn
#pragma unroll
        for (int bi = 0; bi < MB; ++bi)
            if (bj < nb)
                *reinterpret_cast<floatx4 *>(stage + ((wn * 16 + lane % 16) * STAGE_LD + row0 + bi * 16 + 4 * (lane / 16)) * 4) = acc[bj][bi];
        meet();
        Pack<T, PER> now[PASSES];
        static_for<PASSES>([&](auto P) { now[decltype(P)::value] = old[decltype(P)::value]; });
        fetch_old(bj + 1);
        static_for<PASSES>([&](auto P) __attribute__((always_inline)) {
            constexpr int p = decltype(P)::value;
            const int c = piece_c[p], row = piece_row[p], valid = mt - row;
            if (!has(c, bj)) return;
            T *out = C + column(c, bj) * a.ldc + row;
            float v[PER];
#pragma unroll
            for (int h = 0; h < PER / 4; ++h) {
                const floatx4 x = *reinterpret_cast<const floatx4 *>(stage + (c * STAGE_LD + row + 4 * h) * 4);
                v[4 * h] = x.x; v[4 * h + 1] = x.y; v[4 * h + 2] = x.z; v[4 * h + 3] = x.w;
            }
            if (beta != 0.f && valid < PER) {
                if (a.m >= PER) now[p] = __builtin_bit_cast(Pack<T, PER>, shift_elements<T>(__builtin_bit_cast(u32x4, now[p]), PER - valid));
                else now[p] = __builtin_bit_cast(Pack<T, PER>, gather_chunk<T>(out, valid));
            }
            Pack<T, PER> o;
#pragma unroll
            for (int e = 0; e < PER; ++e)
                o.v[e] = static_cast<T>(beta != 0.f ? fmaf(beta, static_cast<float>(now[p].v[e]), alpha * v[e]) : alpha * v[e]);
            if (valid >= PER) *reinterpret_cast<Pack<T, PER> *>(out) = o;
            else store_first<T>(out, o, valid);
        });
    });
}

template <typename T, int WM, int WN, int MB, int NB, bool A_KC, bool B_KC> struct TileBatchConfig {
    static constexpr int DTYPE = sizeof(T) == 4 ? MG_F32 : MG_F16;
    static constexpr int TEAM = WM * WN, TM = WM * MB * 16, TN = WN * NB * 16;
    static bool legal(const BatchedProblem &p)
    {
        if (p.dtype != DTYPE || p.a_trans != A_KC || p.b_trans == B_KC) return false;
        if (TEAM == 1 && (p.m > TM || p.n > TN)) return false;
        return ceil_div(p.m, TM) * ceil_div(p.n, TN) < (int64_t(1) << 31);
    }
    static hipError_t launch(const BatchedProblem &p)
    {
        const int64_t tiles_m = ceil_div(p.m, TM), tiles = tiles_m * ceil_div(p.n, TN);
        TileBatchArgs a{p.A, p.B, p.C, p.a_off, p.b_off, p.c_off, p.alphas, p.betas, p.lda, p.ldb, p.ldc,
                        static_cast<int>(p.m), static_cast<int>(p.n), static_cast<int>(p.k), batchwalk::divisor(tiles_m),
                        0, 0, {}, p.strided ? 1 : 0, p.stride_a, p.stride_b, p.stride_c, p.alpha, p.beta};
        hipError_t e = hipSuccess;
        batchwalk::for_pieces(p.batch, tiles, TEAM == 1 ? 4 : 0, [&](int64_t inst0, int64_t count, int64_t tile0, int64_t piece_tiles) {
            if (p.strided) {
                a.A = static_cast<const T *>(p.A) + inst0 * p.stride_a;
                a.B = static_cast<const T *>(p.B) + inst0 * p.stride_b;
                a.C = static_cast<T *>(p.C) + inst0 * p.stride_c;
            } else {
                a.a_off = p.a_off + inst0;
                a.b_off = p.b_off + inst0;
                a.c_off = p.c_off + inst0;
                a.alphas = p.alphas + inst0;
                a.betas = p.betas + inst0;
            }
            a.batch = count;
            a.tile0 = static_cast<uint32_t>(tile0);
            a.walk = batchwalk::walk(count, piece_tiles);
            const int64_t groups = TEAM == 1 ? ceil_div(count, 4) : batchwalk::work_groups(count, piece_tiles);
            hipLaunchKernelGGL((batched_tile_kernel<T, WM, WN, MB, NB, A_KC, B_KC>), dim3(static_cast<unsigned>(groups)), dim3(256), 0,
                               p.stream, a);
            e = hipGetLastError();
            return e == hipSuccess;
        });
        return e;
    }
    static KernelEntry entry(const char *name)
    {
        mg_config c{};
        c.family = MG_FAMILY_BATCHED;
        c.dtype = DTYPE;
        c.tile_m = TM; c.tile_n = TN; c.tile_k = 128 / static_cast<int>(sizeof(T));
        c.waves_m = WM; c.waves_n = WN;
        c.split_k = 1;
        c.threads = 256;
        c.lds_bytes = TileLds<T, WM, WN, MB, NB, A_KC, B_KC>::BYTES;
        return KernelEntry{name, c, nullptr, nullptr, nullptr, legal, launch};
    }
};

#define MG_TILE_BATCH_REGISTER(table, T, tag, WM, WN, MB, NB)                                     \
    table.push_back(TileBatchConfig<T, WM, WN, MB, NB, false, true>::entry(tag "_mk"));           \
    table.push_back(TileBatchConfig<T, WM, WN, MB, NB, true, true>::entry(tag "_kk"));            \
    table.push_back(TileBatchConfig<T, WM, WN, MB, NB, false, false>::entry(tag "_mn"));          \
    table.push_back(TileBatchConfig<T, WM, WN, MB, NB, true, false>::entry(tag "_kn"));

}  // namespace

void register_batched_tile(std::vector<KernelEntry> &table)
{
    MG_TILE_BATCH_REGISTER(table, float, "batched_tile_32x32", 1, 1, 2, 2)
    MG_TILE_BATCH_REGISTER(table, float, "batched_tile_32x64", 2, 2, 1, 2)
    MG_TILE_BATCH_REGISTER(table, float, "batched_tile_64x64", 2, 2, 2, 2)
    MG_TILE_BATCH_REGISTER(table, _Float16, "hbatched_tile_32x32", 1, 1, 2, 2)
    MG_TILE_BATCH_REGISTER(table, _Float16, "hbatched_tile_32x64", 2, 2, 1, 2)
    MG_TILE_BATCH_REGISTER(table, _Float16, "hbatched_tile_64x64", 2, 2, 2, 2)
}

}  // namespace mg
