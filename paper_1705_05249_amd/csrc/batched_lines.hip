// Batched GEMM, one whole instance per team of one, four or eight wavefronts: both operands are brought to LDS line by line at once, whatever
// their sizes, strides and alignment; then every wavefront takes blocks of 16 columns of C.  FP32, and FP16 storage with FP32 accumulation.
//
// What bounds it: bytes in flight, and the instructions around them.  The kernel of batched_tile.hip spends 370 vector and 280 scalar instructions per
// wavefront of each of its 64 x 64 tiles; 68^3 in FP16 takes four such tiles and two chunks of k.  So here:
//   * nothing is done twice: one team per instance, no chunks, all of k in LDS, where a lane's pieces lie is worked out once per work-group;
//   * work-groups stay and walk over the instances; the next instance's operands are on their way to registers during the products of the
//     current one (without that 68^3 86 us, with it 55: a few resident work-groups cannot hide a memory latency per instance);
//   * a line (a row along k, or a line of rows) is cut into 16-byte pieces from its first element on, and every piece is loaded whole: what
//     runs past the line's end lands in the LDS padding behind it, and a piece that would run past the matrix is loaded as the 16 bytes that end
//     with it and moved down (the matrix has 16 bytes or more); the pieces of C too;
//   * nothing is zeroed: rows that do not exist reach rows and columns of C that do not exist, values of k that do not are masked out of both
//     fragments of the last step of 16 (what LDS holds there may be NaN);
//   * all address arithmetic but the instance's base is 32 bits wide;
//   * results turn through LDS of the wavefront's own, two blocks at a time, and leave as 16-byte pieces, the ends of columns as 8, 4 and 2 bytes.
// us, the kernels before / this (traffic at 6.5 TB/s): FP16 7141 x 68^3 with odd strides 124 / 55 (41), 19400 x 36^3 63 / 39 (23), 8456 x (13, 103, 8) 65 / 22 (9),
// 3660 x 103^3 70 / 55 (36); FP32 7608 x 71^3 202 / 145 (94), 10300 x (22, 122, 9) 72 / 48 (42), 7118 x (152, 8, 8) 63 / 27 (16); over 4000 random calls of 8 to 160 in an
// extent, those not taken included, FP16 0.83 (3.8 % of them more than 5 % slower, up to 1.26) and FP32 0.94 (1.1 %, up to 1.17) of the time.  Eight pieces per lane and operand, for instances of up to 128^3 in FP32, lose to the tiles (86^3 226 / 188): one work-group per compute unit.
// LDS: lines of an operand along k are an odd number of 16 bytes apart (fragments of 16 rows x 8 or 16 bytes touch every bank equally often), lines along
// the rows too (FP32: four reads of 16 consecutive floats at lines 4g, 16 banks apart), or an odd number of 32 bytes (FP16: transposing reads).
#include "mfma_any_kernel.h"

namespace mg {
namespace {

typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));

struct LinesOperand {
    const void *X;
    const int64_t *off;
    int64_t stride;
    int32_t ld;
    int32_t pieces;                // of the operand,
    int32_t per_line, magic;       // and of a line; idx / per_line = idx * magic >> LINES_SHIFT
    int32_t last;                  // the last element that 16 bytes of the operand start from
    int32_t pitch;                 // bytes between lines in LDS
};
struct LinesArgs {
    LinesOperand a, b;
    void *C;
    const int64_t *c_off;
    const float *alphas, *betas;
    int64_t stride_c;
    uint32_t batch;
    int32_t ldc, m, n, k;
    int32_t b_lds, stage_lds, team_lds;      // LDS: op(A), op(B), the wavefronts' strips; bytes of a team
    int32_t groups, rows_per_group;          // groups of row blocks (rows_per_group blocks of 16)
    int strided;
    float alpha, beta;
};
constexpr int LINES_SHIFT = 19, LINES_CUS = 256;
constexpr int LINES_LDS = 80 * 1024;          // of a work-group: two per compute unit

// fragment of 16 rows x 16 values of k: lane (r, g) holds X[r][4g + s], s = 0..3
template <typename T> struct LinesFragment;
template <> struct LinesFragment<float> { using type = floatx4; };
template <> struct LinesFragment<_Float16> { using type = halfx4; };

template <typename T, bool KCONTIG> struct LinesReader {
    using Frag = typename LinesFragment<T>::type;
    // lane's address of row 0, k 0
    static __device__ __forceinline__ int base(int lane, int pitch)
    {
        const int r = lane % 16, g = lane / 16;
        if constexpr (KCONTIG) return r * pitch + g * 4 * static_cast<int>(sizeof(T));
        else if constexpr (sizeof(T) == 4) return 4 * g * pitch + r * 4;
        else return (4 * g + r / 4) * pitch + 8 * (r % 4);
    }
    static __device__ __forceinline__ int row_step(int pitch) { return KCONTIG ? 16 * pitch : 16 * static_cast<int>(sizeof(T)); }
    static __device__ __forceinline__ int k_step(int pitch) { return KCONTIG ? 16 * static_cast<int>(sizeof(T)) : 16 * pitch; }
    static __device__ __forceinline__ Frag read(const char *p, int pitch)
    {
        if constexpr (KCONTIG) return *reinterpret_cast<const Frag *>(p);
        else if constexpr (sizeof(T) == 4)
            return Frag{*reinterpret_cast<const float *>(p), *reinterpret_cast<const float *>(p + pitch), *reinterpret_cast<const float *>(p + 2 * pitch),
                        *reinterpret_cast<const float *>(p + 3 * pitch)};
        else {
#if defined(__HIP_DEVICE_COMPILE__)
            return __builtin_bit_cast(Frag, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4 *)p));
#else
            return Frag{};
#endif
        }
    }
};

// the values of k behind the sum's end: `left` of the lane's four exist
__device__ __forceinline__ floatx4 keep_first(floatx4 v, int left)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = e < left ? v[e] : 0.f;
    return v;
}
__device__ __forceinline__ halfx4 keep_first(halfx4 v, int left)
{
    u32x2 w = __builtin_bit_cast(u32x2, v);
    w.x = left >= 2 ? w.x : (left == 1 ? w.x & 0xffffu : 0u);
    w.y = left >= 4 ? w.y : (left == 3 ? w.y & 0xffffu : 0u);
    return __builtin_bit_cast(halfx4, w);
}
__device__ __forceinline__ void lines_mma(floatx4 &c, halfx4 x, halfx4 y) { c = __builtin_amdgcn_mfma_f32_16x16x16f16(x, y, c, 0, 0, 0); }
template <int N> __device__ __forceinline__ void lines_step(floatx4 (&c)[N], const floatx4 (&x)[N], floatx4 y)
{
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < N; ++i) c[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i][e], y[e], c[i], 0, 0, 0);
}
template <int N> __device__ __forceinline__ void lines_step(floatx4 (&c)[N], const halfx4 (&x)[N], halfx4 y)
{
#pragma unroll
    for (int i = 0; i < N; ++i) lines_mma(c[i], x[i], y);
}

// An operand's pieces tid + i * NT, i < U, to registers, and from there to LDS
template <typename T, int NT, int U> struct LinesLoader {
    static constexpr int V = 16 / static_cast<int>(sizeof(T));
    u32x4 regs[U];
    uint32_t from[U];              // byte of the operand
    int at[U];                     // LDS byte | elements to move down (at most 7)
    __device__ __forceinline__ void prepare(const LinesOperand &o, int lds, int tid)
    {
        static_for<U>([&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            const int idx = min(tid + i * NT, o.pieces - 1);                    // (a lane beyond the last piece repeats it)
            const int line = static_cast<int>(__umul24(idx, o.magic) >> LINES_SHIFT), piece = idx - __mul24(line, o.per_line);
            const int wanted = __mul24(line, o.ld) + piece * V, first = min(wanted, o.last);
            at[i] = (lds + __mul24(line, o.pitch) + piece * 16) | (wanted - first);
            from[i] = static_cast<uint32_t>(first) * static_cast<uint32_t>(sizeof(T));
            // (kept, not worked out again for every instance)
            asm volatile("" : "+v"(at[i]), "+v"(from[i]));
        });
    }
    __device__ __forceinline__ void load(const LinesOperand &o, const char *base)
    {
        static_for<U>([&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            if (i * NT < o.pieces) regs[i] = load_unaligned_chunk<T>(reinterpret_cast<const T *>(base + from[i]));
        });
    }
    __device__ __forceinline__ void store(const LinesOperand &o, char *lds)
    {
        static_for<U>([&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            if (i * NT >= o.pieces) return;
            int to = at[i];
            asm volatile("" : "+v"(to));                                        // (else the masks of all lanes to move are kept, and spilled)
            if (to & 7) regs[i] = shift_elements<T>(regs[i], to & 7);
            *reinterpret_cast<u32x4 *>(lds + (to & ~15)) = regs[i];
        });
    }
};

// Row blocks of a group, and the strip that a wavefront's results turn through
constexpr int LINES_G = 2, STRIP_LD = LINES_G * 16 + 4, STRIP = 16 * STRIP_LD * 4;      // (floats per column; bytes)

// TEAM: wavefronts per instance; U: pieces of each operand that a lane holds of the instance to come.  A team of one shares its work-group with
// three others.  Work-groups stay and walk over the instances.
template <typename T, int TEAM, int U, bool A_KC, bool B_KC>
__global__ __launch_bounds__(TEAM == 8 ? 512 : 256, 4) void batched_lines_kernel(const LinesArgs a)
{
    constexpr int NT = TEAM * 64, TEAMS = TEAM == 1 ? 4 : 1, V = 16 / static_cast<int>(sizeof(T)), G = LINES_G;
    constexpr int PER_COL = G * 16 / V, COLS = 64 / PER_COL, PASSES = 16 / COLS;           // 16-byte pieces of a column of a strip, columns of a pass
    using ReadA = LinesReader<T, A_KC>;
    using ReadB = LinesReader<T, B_KC>;
    using Frag = typename LinesFragment<T>::type;
    extern __shared__ __attribute__((aligned(16))) char shared[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int tid = TEAM == 1 ? lane : static_cast<int>(threadIdx.x);
    char *lds = shared + (TEAM == 1 ? wave * a.team_lds : 0);
    auto meet = [] {
        if constexpr (TEAM == 1) {
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            lds_barrier();
        }
    };

    struct Instance {
        float alpha, beta;
        const char *A, *B;
        char *C;
    };
    auto find = [&](uint32_t i) __attribute__((always_inline)) {
        const int64_t at_a = a.strided ? i * a.a.stride : a.a.off[i], at_b = a.strided ? i * a.b.stride : a.b.off[i], at_c = a.strided ? i * a.stride_c : a.c_off[i];
        return Instance{a.strided ? a.alpha : a.alphas[i], a.strided ? a.beta : a.betas[i], static_cast<const char *>(a.a.X) + at_a * static_cast<int64_t>(sizeof(T)),
                        static_cast<const char *>(a.b.X) + at_b * static_cast<int64_t>(sizeof(T)), static_cast<char *>(a.C) + at_c * static_cast<int64_t>(sizeof(T))};
    };
    const uint32_t stride = gridDim.x * TEAMS;
    uint32_t inst = TEAM == 1 ? blockIdx.x * 4 + wave : blockIdx.x;
    if (inst >= a.batch) return;
    Instance it = find(inst);
    LinesLoader<T, NT, U> la, lb;
    la.prepare(a.a, 0, tid);
    lb.prepare(a.b, a.b_lds, tid);
    if (it.alpha != 0.f) {                                         // alpha == 0: A and B are not read at all
        la.load(a.a, it.A);
        lb.load(a.b, it.B);
    }
    const int base_a = ReadA::base(lane, a.a.pitch), base_b = a.b_lds + ReadB::base(lane, a.b.pitch);
    const int step_a = ReadA::k_step(a.a.pitch), step_b = ReadB::k_step(a.b.pitch), rows_a = ReadA::row_step(a.a.pitch), rows_b = ReadB::row_step(a.b.pitch);
    char *strip = lds + a.stage_lds + (TEAM == 1 ? 0 : wave * STRIP);
    char *strip_in = strip + ((lane % 16) * STRIP_LD + 4 * (lane / 16)) * 4;
    const char *strip_out = strip + (lane / PER_COL * STRIP_LD + lane % PER_COL * V) * 4;

    for (;;) {
        const bool more = inst + stride < a.batch;                     // (fewer than 2^31 instances)
        const Instance next = find(more ? inst + stride : inst);
        const float alpha = it.alpha, beta = it.beta;
        char *C = it.C;
        const int k = alpha == 0.f ? 0 : a.k;
        if (k > 0) {
            la.store(a.a, lds);
            lb.store(a.b, lds);
        }
        meet();
        if (more && next.alpha != 0.f) {
            la.load(a.a, next.A);
            lb.load(a.b, next.B);
        }
        const int steps = (k + 15) / 16, left = k - (steps - 1) * 16 - 4 * (lane / 16);         // values of the last step that this lane has

        // units: a group of row blocks of a block of columns; which wavefront starts where changes from instance to instance
        int group = TEAM == 1 ? 0 : (wave + static_cast<int>(inst)) & (TEAM - 1), block_col = 0;
        for (;;) {
            while (group >= a.groups) {
                group -= a.groups;
                ++block_col;
            }
            const int col0 = block_col * 16, row0 = group * a.rows_per_group * 16;
            if (col0 >= a.n) break;
            const int rows = min(a.m - row0, a.rows_per_group * 16), blocks = (rows + 15) / 16;

            // this lane's pieces of the unit: rows lane % PER_COL * V .. of every COLS-th column
            // (of a piece that ends beyond the column the 16 bytes that end with it)
            const int row = lane % PER_COL * V, valid = rows - row, beyond = max(V - max(valid, 0), 0);
            u32x4 old[PASSES];
            int place[PASSES];
#pragma unroll
            for (int h = 0; h < PASSES; ++h) {
                const int col = col0 + lane / PER_COL + COLS * h;
                place[h] = __mul24(col, a.ldc) + row0 + row;
                if (beta != 0.f && col < a.n && valid > 0 && a.m >= V)
                    old[h] = load_unaligned_chunk<T>(reinterpret_cast<const T *>(C + static_cast<uint32_t>(place[h] - beyond) * static_cast<uint32_t>(sizeof(T))));
            }

            auto unit = [&](auto N) __attribute__((always_inline)) {
                constexpr int n = decltype(N)::value;
                floatx4 acc[n];
#pragma unroll
                for (int i = 0; i < n; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
                const char *pa = lds + base_a + group * a.rows_per_group * rows_a, *pb = lds + base_b + block_col * rows_b;
                Frag x[n], y;
                for (int s = 1; s < steps; ++s) {
                    y = ReadB::read(pb, a.b.pitch);
#pragma unroll
                    for (int i = 0; i < n; ++i) x[i] = ReadA::read(pa + i * rows_a, a.a.pitch);
                    lines_step<n>(acc, x, y);
                    pa += step_a;
                    pb += step_b;
                }
                if (steps > 0) {
                    y = keep_first(ReadB::read(pb, a.b.pitch), left);
#pragma unroll
                    for (int i = 0; i < n; ++i) x[i] = keep_first(ReadA::read(pa + i * rows_a, a.a.pitch), left);
                    lines_step<n>(acc, x, y);
                }
#pragma unroll
                for (int i = 0; i < n; ++i) *reinterpret_cast<floatx4 *>(strip_in + i * 64) = acc[i];
            };
            if (blocks == 1) unit(std::integral_constant<int, 1>{});
            else unit(std::integral_constant<int, G>{});

            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int h = 0; h < PASSES; ++h) {
                if (col0 + lane / PER_COL + COLS * h >= a.n || valid <= 0) continue;
                T *out = reinterpret_cast<T *>(C + static_cast<uint32_t>(place[h]) * static_cast<uint32_t>(sizeof(T)));
                if (beta != 0.f && beyond > 0) {
                    if (a.m >= V) old[h] = shift_elements<T>(old[h], beyond);
                    else old[h] = gather_chunk<T>(out, valid);
                }
                const Pack<T, V> was = __builtin_bit_cast(Pack<T, V>, old[h]);
                Pack<T, V> o;
                const char *from = strip_out + h * COLS * STRIP_LD * 4;
#pragma unroll
                for (int q = 0; q < V / 4; ++q) {
                    const floatx4 v = *reinterpret_cast<const floatx4 *>(from + 16 * q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float r = alpha * v[e];
                        if (beta != 0.f) r = fmaf(beta, static_cast<float>(was.v[4 * q + e]), r);
                        o.v[4 * q + e] = static_cast<T>(r);
                    }
                }
                if (valid >= V) *reinterpret_cast<Pack<T, V> *>(out) = o;
                else store_first<T>(out, o, valid);
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");       // (the strip is read before the next unit writes it)
            __builtin_amdgcn_wave_barrier();
            group += TEAM;
        }
        if (!more) break;
        meet();                                                        // everyone is done with this instance's operands
        inst += stride;
        it = next;
    }
}

// host: the lines of an operand of `rows` rows and k values, false where the kernel does not take it
template <typename T> bool plan_operand(LinesOperand &o, int64_t rows, int64_t k, int64_t ld, bool kcontig, int64_t &lds_bytes)
{
    constexpr int V = 16 / static_cast<int>(sizeof(T));
    const int64_t length = kcontig ? k : rows, lines = kcontig ? rows : k;
    if (length > 4096 || lines > 2048 || ld >= (int64_t(1) << 20)) return false;
    const int64_t per = ceil_div(length, V), span = (lines - 1) * ld + length;
    if (span < V || span >= (int64_t(1) << 29) || lines * per * per >= (int64_t(1) << LINES_SHIFT) || lines * per >= 8192) return false;
    const int64_t row_bytes = ceil_div(length, 16) * 16 * static_cast<int64_t>(sizeof(T));  // whole blocks of 16
    int64_t pitch = row_bytes > per * 16 ? row_bytes : per * 16;
    if (!kcontig && sizeof(T) == 2) pitch = (pitch / 32 | 1) * 32;                          // (row_bytes is a multiple of 32)
    else pitch = (pitch / 16 | 1) * 16;
    o.ld = static_cast<int32_t>(ld);
    o.pieces = static_cast<int32_t>(lines * per);
    o.per_line = static_cast<int32_t>(per);
    o.magic = static_cast<int32_t>(((int64_t(1) << LINES_SHIFT) + per - 1) / per);
    o.last = static_cast<int32_t>(span - V);
    o.pitch = static_cast<int32_t>(pitch);
    lds_bytes = ceil_div(lines, 16) * 16 * pitch;
    return true;
}

template <typename T, int TEAM, int U> bool plan_lines(const BatchedProblem &p, LinesArgs &a)
{
    if (p.k < 1 || p.m > 1024 || p.n > 1024 || p.ldc >= (int64_t(1) << 20) || p.n * p.ldc >= (int64_t(1) << 29)) return false;
    int64_t bytes_a = 0, bytes_b = 0;
    if (!plan_operand<T>(a.a, p.m, p.k, p.lda, p.a_trans, bytes_a) || !plan_operand<T>(a.b, p.n, p.k, p.ldb, !p.b_trans, bytes_b)) return false;
    const int64_t bytes = bytes_a + bytes_b + TEAM * STRIP;
    if (a.a.pieces > U * TEAM * 64 || a.b.pieces > U * TEAM * 64 || bytes * (TEAM == 1 ? 4 : 1) > LINES_LDS) return false;
    a.b_lds = static_cast<int32_t>(bytes_a);
    a.stage_lds = static_cast<int32_t>(bytes_a + bytes_b);
    a.team_lds = static_cast<int32_t>(bytes);
    a.ldc = static_cast<int32_t>(p.ldc);
    a.m = static_cast<int32_t>(p.m);
    a.n = static_cast<int32_t>(p.n);
    a.k = static_cast<int32_t>(p.k);
    const int64_t blocks = ceil_div(p.m, 16), groups = ceil_div(blocks, LINES_G);
    // (fewer units than wavefronts: single blocks)
    a.rows_per_group = groups * ceil_div(p.n, 16) < TEAM ? 1 : static_cast<int32_t>(ceil_div(blocks, groups));
    a.groups = static_cast<int32_t>(ceil_div(blocks, a.rows_per_group));
    return true;
}

// work-groups that the chip holds: by their LDS, and four (of eight wavefronts two) of a compute unit by their registers
template <int TEAM> int64_t resident_groups(int64_t group_lds)
{
    constexpr int64_t MOST = TEAM == 8 ? 2 : 4;
    const int64_t fit = 160 * 1024 / group_lds;
    return LINES_CUS * (fit < MOST ? fit : MOST);
}

template <int TEAM> bool shape_of(const BatchedProblem &p, LinesShape *shape)
{
    constexpr int TEAMS = TEAM == 1 ? 4 : 1;
    LinesArgs a{};
    if (!plan_lines<float, TEAM, 4>(p, a)) return false;
    shape->pieces = a.a.pieces + a.b.pieces;
    shape->resident = resident_groups<TEAM>(a.team_lds * TEAMS) * TEAMS;
    return true;
}

template <typename T, int TEAM, int U, bool A_KC, bool B_KC> struct LinesConfig {
    static constexpr int DTYPE = sizeof(T) == 4 ? MG_F32 : MG_F16, TEAMS = TEAM == 1 ? 4 : 1;
    static bool legal(const BatchedProblem &p)
    {
        LinesArgs a;
        return p.dtype == DTYPE && p.a_trans == A_KC && p.b_trans != B_KC && plan_lines<T, TEAM, U>(p, a);
    }
    static hipError_t launch(const BatchedProblem &p)
    {
        LinesArgs a{};
        if (!plan_lines<T, TEAM, U>(p, a)) return hipErrorInvalidValue;
        auto kernel = batched_lines_kernel<T, TEAM, U, A_KC, B_KC>;
        static bool attr_set = false;   // raising the dynamic LDS limit is idempotent; races are harmless
        if (!attr_set) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, LINES_LDS);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        a.strided = p.strided ? 1 : 0;
        a.alpha = p.alpha;
        a.beta = p.beta;
        a.a.stride = p.stride_a;
        a.b.stride = p.stride_b;
        a.stride_c = p.stride_c;
        const int64_t group_lds = a.team_lds * TEAMS, resident = resident_groups<TEAM>(group_lds);
        hipError_t e = hipSuccess;
        constexpr int64_t MOST = int64_t(1) << 30;
        for (int64_t inst0 = 0; inst0 < p.batch && e == hipSuccess; inst0 += MOST) {
            const int64_t count = p.batch - inst0 < MOST ? p.batch - inst0 : MOST;
            a.a.X = static_cast<const T *>(p.A) + (p.strided ? inst0 * p.stride_a : 0);
            a.b.X = static_cast<const T *>(p.B) + (p.strided ? inst0 * p.stride_b : 0);
            a.C = static_cast<T *>(p.C) + (p.strided ? inst0 * p.stride_c : 0);
            if (!p.strided) {
                a.a.off = p.a_off + inst0;
                a.b.off = p.b_off + inst0;
                a.c_off = p.c_off + inst0;
                a.alphas = p.alphas + inst0;
                a.betas = p.betas + inst0;
            }
            a.batch = static_cast<uint32_t>(count);
            const int64_t groups = ceil_div(count, TEAMS);
            hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(groups < resident ? groups : resident)), dim3(TEAM == 8 ? 512 : 256),
                               static_cast<unsigned>(group_lds), p.stream, a);
            e = hipGetLastError();
        }
        return e;
    }
    static KernelEntry entry(const char *name)
    {
        mg_config c{};
        c.family = MG_FAMILY_BATCHED;
        c.dtype = DTYPE;
        c.tile_m = c.tile_n = 16;
        c.tile_k = 16;
        c.waves_m = 1;
        c.waves_n = TEAM;
        c.split_k = 1;
        c.threads = TEAM == 8 ? 512 : 256;
        c.lds_bytes = LINES_LDS;
        return KernelEntry{name, c, nullptr, nullptr, nullptr, legal, launch};
    }
};

#define MG_LINES(T, TEAM, U, tag)                                                   \
    table.push_back(LinesConfig<T, TEAM, U, false, true>::entry(tag "_mk"));        \
    table.push_back(LinesConfig<T, TEAM, U, true, true>::entry(tag "_kk"));         \
    table.push_back(LinesConfig<T, TEAM, U, false, false>::entry(tag "_mn"));       \
    table.push_back(LinesConfig<T, TEAM, U, true, false>::entry(tag "_kn"));

}  // namespace

bool batched_lines_shape(const BatchedProblem &p, int team, LinesShape *shape)
{
    switch (team) {
    case 1: return shape_of<1>(p, shape);
    case 4: return shape_of<4>(p, shape);
    default: return shape_of<8>(p, shape);
    }
}

void register_batched_lines(std::vector<KernelEntry> &table)
{
    MG_LINES(float, 1, 4, "batched_lines_w1")
    MG_LINES(float, 4, 4, "batched_lines_w4")
    MG_LINES(float, 8, 4, "batched_lines_w8")
    MG_LINES(_Float16, 1, 4, "hbatched_lines_w1")
    MG_LINES(_Float16, 4, 4, "hbatched_lines_w4")
    MG_LINES(_Float16, 8, 4, "hbatched_lines_w8")
}

}  // namespace mg
