// m == 1 or n == 1: the product is a matrix-vector product, bound by reading the matrix once
// from HBM (the paper treats GEMV as the bandwidth-bound level-2 representative, Section 4.2;
// here it is the skinny corner of GEMM).
//
//      out[o] = alpha * sum_l Mat(o, l) * vec[l] + beta * out[o]
//
//   n == 1:  Mat = op(A) (o = row i),  vec = column 0 of op(B),  out = column 0 of C
//   m == 1:  Mat = op(B)^T (o = column j),  vec = row 0 of op(A),  out = row 0 of C
//
// Kernels by how the matrix lies in memory:
//   dot   Mat(o, .) contiguous along l: one wavefront per output (four outputs when there are
//         thousands of them), lanes stride over l with 16-byte loads (issued at element alignment:
//         rows of a padded matrix are not 16-byte aligned), cross-lane sum at the end;
//   axpy  Mat(., l) contiguous along o: a work-group owns 64 x (16 bytes / element size)
//         consecutive outputs, each lane a 16-byte run of them; its four wavefronts take
//         l = w, w+4, ... with eight loads in flight per lane and meet in LDS;
//   panel the same order, with a work-group on fewer outputs and more of the sum.
// Outputs that end inside a lane's run (axpy, panel): the run is taken as the V outputs that end with the last one and its first elements dropped, so
// that every lane loads 16 bytes, eight columns in flight (element by element that one lane's column loop set the time of the call; us, before / now:
// FP16 1518 outputs of 8038 terms 17.7 / 9.2, 5003 of 10368 39 / 24, FP32 14419 of 5564 88 / 55; 0.85 over 128 ragged calls; others have flavours without, 1 % faster).
// What such a call of a few microseconds pays for it is kept below 0.2 us: every lane stores its run with the same masked stores (two ways of
// storing, one per kind of lane, took FP16 9 x 15 from 2.8 to 3.1 us; now 2.9).
// Few outputs and a long sum leave most compute units idle, so both kernels can cut the sum into
// `split` slices (grid.y): each slice writes FP32 partial sums to the workspace and a small
// second kernel adds them and applies alpha and beta.
#include <type_traits>

#include "internal.h"

namespace mg {
namespace {

template <typename T, int V> struct __attribute__((packed, aligned(sizeof(T)))) PackedVec {
    T v[V];
};

// 16 bytes of the matrix at element alignment, as a streaming (non-temporal) load: every matrix element is
// used once, and a read stream marked this way runs about 10 % faster on this part than a plain one
// (7.1 against 6.3-6.5 TB/s for a 2 GiB buffer).
template <typename T, int V> __device__ inline PackedVec<T, V> stream_load(const T *p)
{
    typedef T Wide __attribute__((ext_vector_type(V)));
    typedef Wide Unaligned __attribute__((aligned(sizeof(T))));
    const Wide w = __builtin_nontemporal_load(reinterpret_cast<const Unaligned *>(p));
    PackedVec<T, V> r;
#pragma unroll
    for (int e = 0; e < V; ++e) r.v[e] = w[e];
    return r;
}

__device__ inline float wave_sum(float x)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

template <typename T> __device__ inline void finish(T *p, float sum, float alpha, float beta)
{
    float v = alpha * sum;
    if (beta != 0.f) v = fmaf(beta, static_cast<float>(*p), v);
    *p = static_cast<T>(v);
}

// partial != nullptr: slice blockIdx.y of the sum goes to partial[blockIdx.y * outputs + o] unscaled.
// R: rows per wavefront.  With many rows a wavefront takes four at once: their loads are in flight
// together (a short row is a single round of loads) and each piece of the vector is fetched once for four rows.
template <typename T, int R>
__global__ __launch_bounds__(256) void gemv_dot_kernel(int64_t outputs, int64_t k, int64_t k_per_split,
                                                        const T *__restrict__ mat, int64_t stride_o,
                                                        const T *__restrict__ vec, int64_t stride_v,
                                                        T *__restrict__ out, int64_t stride_out,
                                                        float *__restrict__ partial, float alpha, float beta)
{
    constexpr int V = 16 / static_cast<int>(sizeof(T));
    using Vec = PackedVec<T, V>;
    const int64_t o0 = (static_cast<int64_t>(blockIdx.x) * 4 + threadIdx.x / 64) * R;
    if (o0 >= outputs) return;
    const int lane = threadIdx.x % 64;
    const int64_t k0 = static_cast<int64_t>(blockIdx.y) * k_per_split;
    const int64_t k1 = k0 + k_per_split < k ? k0 + k_per_split : k;
    const T *__restrict__ row[R];
    float acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        // rows past the end repeat the last one: loaded, never stored
        row[r] = mat + (o0 + r < outputs ? o0 + r : outputs - 1) * stride_o;
        acc[r] = 0.f;
    }
    int64_t l = k0;
    if (stride_v == 1 && k1 > k0) {
        auto piece = [&](int64_t at) {
            Vec a[R];
#pragma unroll
            for (int r = 0; r < R; ++r) a[r] = stream_load<T, V>(row[r] + at);
            const Vec b = *reinterpret_cast<const Vec *>(vec + at);
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int e = 0; e < V; ++e)
                    acc[r] = fmaf(static_cast<float>(a[r].v[e]), static_cast<float>(b.v[e]), acc[r]);
        };
        // whole rounds of 64 pieces of 16 bytes (the same count for every lane, so the loop unrolls with
        // its loads up front), then the pieces of a last partial round; what is left is shorter than a piece
        const int64_t rounds_end = k1 - (k1 - k0) % (64 * V);
        if constexpr (R == 1) {
#pragma unroll 4
            for (l = k0 + static_cast<int64_t>(lane) * V; l < rounds_end; l += 64 * V) piece(l);
        } else {
#pragma unroll 2
            for (l = k0 + static_cast<int64_t>(lane) * V; l < rounds_end; l += 64 * V) piece(l);
        }
        l = rounds_end + static_cast<int64_t>(lane) * V;
        if (l + V <= k1) piece(l);
        l = k1 - (k1 - k0) % V;
    }
    for (l += lane; l < k1; l += 64) {
        const float x = static_cast<float>(vec[l * stride_v]);
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = fmaf(static_cast<float>(row[r][l]), x, acc[r]);
    }
    float mine = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float s = wave_sum(acc[r]);
        if (lane == r) mine = s;
    }
    if (lane < R && o0 + lane < outputs) {
        if (partial != nullptr) partial[static_cast<int64_t>(blockIdx.y) * outputs + o0 + lane] = mine;
        else finish(out + (o0 + lane) * stride_out, mine, alpha, beta);
    }
}

// Where the outputs end: with a lane's run of V, inside one, or (FP16) inside the first.  A flavour for FP16 calls of fewer than eight outputs: the masked stores of
// the second cost them 0.2 of 3.6 us; FP32 ones of fewer than four lose as much to the element loop by itself (2 outputs of 2487 terms 4.8 / 5.5 us).
enum class Ends { whole, ragged, few };
template <typename T> Ends ends_of(int64_t outputs)
{
    constexpr int64_t V = 16 / static_cast<int>(sizeof(T));
    return sizeof(T) == 2 && outputs < V ? Ends::few : (outputs % V != 0 ? Ends::ragged : Ends::whole);
}
// fewer than V outputs may come
template <typename T, Ends ENDS> constexpr bool SHORT_RUN = ENDS == Ends::few || (ENDS == Ends::ragged && sizeof(T) == 4);

template <typename T, Ends ENDS>
__global__ __launch_bounds__(256) void gemv_axpy_kernel(int64_t outputs, int64_t k, int64_t k_per_split,
                                                         const T *__restrict__ mat, int64_t stride_l,
                                                         const T *__restrict__ vec, int64_t stride_v,
                                                         T *__restrict__ out, int64_t stride_out,
                                                         float *__restrict__ partial, float alpha, float beta)
{
    constexpr int V = 16 / static_cast<int>(sizeof(T));
    constexpr int OB = 64 * V;                      // outputs per work-group
    constexpr int U = 8;                            // columns in flight per wavefront (16: no faster)
    using Vec = PackedVec<T, V>;
    __shared__ float part[4][OB];
    const int lane = threadIdx.x % 64;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int64_t first = static_cast<int64_t>(blockIdx.x) * OB;
    const int64_t o = first + lane * V;
    const int64_t k0 = static_cast<int64_t>(blockIdx.y) * k_per_split;
    const int64_t k1 = k0 + k_per_split < k ? k0 + k_per_split : k;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    // a run that ends beyond the outputs is taken as the V outputs that end with them; the first `dropped` are the run's before it
    const int64_t at = ENDS != Ends::ragged || o + V <= outputs ? o : outputs - V;
    const int dropped = ENDS == Ends::ragged && (!SHORT_RUN<T, ENDS> || at >= 0) ? static_cast<int>(o - at) : 0;
    if (ENDS != Ends::few && o < outputs && (!SHORT_RUN<T, ENDS> || at >= 0)) {
        const T *__restrict__ col = mat + at;
        int64_t l = k0 + w;
        for (; l + 4 * (U - 1) < k1; l += 4 * U) {
            Vec a[U];
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u] = stream_load<T, V>(col + (l + 4 * u) * stride_l);
                x[u] = static_cast<float>(vec[(l + 4 * u) * stride_v]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int e = 0; e < V; ++e) acc[e] = fmaf(static_cast<float>(a[u].v[e]), x[u], acc[e]);
        }
        for (; l < k1; l += 4) {
            const Vec a = stream_load<T, V>(col + l * stride_l);
            const float x = static_cast<float>(vec[l * stride_v]);
#pragma unroll
            for (int e = 0; e < V; ++e) acc[e] = fmaf(static_cast<float>(a.v[e]), x, acc[e]);
        }
    } else if (SHORT_RUN<T, ENDS> && o < outputs) {
        // element by element
        for (int64_t l = k0 + w; l < k1; l += 4) {
            const float x = static_cast<float>(vec[l * stride_v]);
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (o + e < outputs) acc[e] = fmaf(static_cast<float>(mat[o + e + l * stride_l]), x, acc[e]);
        }
    }
#pragma unroll
    for (int e = 0; e < V; ++e)
        if (ENDS != Ends::ragged || e >= dropped) part[w][lane * V + e - dropped] = acc[e];
    __syncthreads();
    for (int i = threadIdx.x; i < OB; i += 256) {
        const int64_t oo = first + i;
        if (oo >= outputs) break;
        const float s = (part[0][i] + part[1][i]) + (part[2][i] + part[3][i]);
        if (partial != nullptr) partial[static_cast<int64_t>(blockIdx.y) * outputs + oo] = s;
        else finish(out + oo * stride_out, s, alpha, beta);
    }
}

// axpy order with few outputs: the kernel above gives a work-group 64 x 16 bytes of outputs, so 4096 of them make sixteen work-groups
// and the sum must be cut into slices, with partial sums through memory and a second launch.  Here LR lanes side by side take a
// run of LR x 16 bytes of a column, the other 64 / LR lanes of the wavefront the next columns, and sixteen wavefronts share
// the sum of one work-group; lanes, then wavefronts (through LDS), are added at the end.
// STREAM: non-temporal loads, see gemv_launch.
template <typename T, int LR, bool STREAM, Ends ENDS>
__global__ __launch_bounds__(1024) void gemv_panel_kernel(int64_t outputs, int64_t k, int64_t k_per_split,
                                                           const T *__restrict__ mat, int64_t stride_l,
                                                           const T *__restrict__ vec, int64_t stride_v,
                                                           T *__restrict__ out, int64_t stride_out,
                                                           float *__restrict__ partial, float alpha, float beta)
{
    constexpr int V = 16 / static_cast<int>(sizeof(T));
    constexpr int OB = LR * V;                      // outputs per work-group
    constexpr int CL = 64 / LR;                     // columns per wavefront and load instruction
    constexpr int WAVES = 16;
    constexpr int U = 8;                            // load instructions in flight per wavefront
    constexpr int STEP = WAVES * CL;
    using Vec = PackedVec<T, V>;
    __shared__ float part[WAVES][OB];
    auto load = [](const T *p) {
        if constexpr (STREAM) return stream_load<T, V>(p);
        else return *reinterpret_cast<const Vec *>(p);
    };
    const int lane = threadIdx.x % 64;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    // neighbours in memory on the same XCD: they share cache lines
    const int xcd = blockIdx.x % 8, q = gridDim.x / 8, rem = gridDim.x % 8;
    const int group = xcd * q + (xcd < rem ? xcd : rem) + blockIdx.x / 8;
    const int64_t first = static_cast<int64_t>(group) * OB;
    const int64_t o = first + lane % LR * V;
    const int64_t k0 = static_cast<int64_t>(blockIdx.y) * k_per_split;
    const int64_t k1 = k0 + k_per_split < k ? k0 + k_per_split : k;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    int64_t l = k0 + w * CL + lane / LR;
    // (the last run as in the kernel above)
    const int64_t at = ENDS != Ends::ragged || o + V <= outputs ? o : outputs - V;
    const int dropped = ENDS == Ends::ragged && (!SHORT_RUN<T, ENDS> || at >= 0) ? static_cast<int>(o - at) : 0;
    if (ENDS != Ends::few && o < outputs && (!SHORT_RUN<T, ENDS> || at >= 0)) {
        const T *__restrict__ col = mat + at;
        for (; l + STEP * (U - 1) < k1; l += STEP * U) {
            Vec a[U];
            T x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u] = load(col + (l + STEP * u) * stride_l);
                x[u] = vec[(l + STEP * u) * stride_v];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int e = 0; e < V; ++e) acc[e] = fmaf(static_cast<float>(a[u].v[e]), static_cast<float>(x[u]), acc[e]);
        }
#pragma unroll 2
        for (; l < k1; l += STEP) {
            const Vec a = load(col + l * stride_l);
            const float x = static_cast<float>(vec[l * stride_v]);
#pragma unroll
            for (int e = 0; e < V; ++e) acc[e] = fmaf(static_cast<float>(a.v[e]), x, acc[e]);
        }
    } else if (SHORT_RUN<T, ENDS> && o < outputs) {
        // (likewise)
        for (; l < k1; l += STEP) {
            const float x = static_cast<float>(vec[l * stride_v]);
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (o + e < outputs) acc[e] = fmaf(static_cast<float>(mat[o + e + l * stride_l]), x, acc[e]);
        }
    }
#pragma unroll
    for (int off = LR; off < 64; off *= 2)
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] += __shfl_xor(acc[e], off, 64);
    if (lane < LR) {
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (ENDS != Ends::ragged || e >= dropped) part[w][lane * V + e - dropped] = acc[e];
    }
    __syncthreads();
    const int i = threadIdx.x;
    if (i < OB && first + i < outputs) {
        float s = 0.f;
#pragma unroll
        for (int z = 0; z < WAVES; ++z) s += part[z][i];
        if (partial != nullptr) partial[static_cast<int64_t>(blockIdx.y) * outputs + first + i] = s;
        else finish(out + (first + i) * stride_out, s, alpha, beta);
    }
}

// out[o] <- alpha * sum_z partial[z][o] + beta * out[o]: 16 outputs per work-group, 16 threads share the
// slices of each output
template <typename T>
__global__ __launch_bounds__(256) void gemv_reduce_kernel(const float *__restrict__ partial, int split, int64_t outputs,
                                                           T *__restrict__ out, int64_t stride_out, float alpha,
                                                           float beta)
{
    __shared__ float part[16][17];
    const int oi = threadIdx.x % 16, zl = threadIdx.x / 16;
    const int64_t o = static_cast<int64_t>(blockIdx.x) * 16 + oi;
    float s = 0.f;
    if (o < outputs) {
#pragma unroll 4
        for (int z = zl; z < split; z += 16) s += partial[z * outputs + o];
    }
    part[zl][oi] = s;
    __syncthreads();
    if (zl == 0 && o < outputs) {
        float t = 0.f;
#pragma unroll
        for (int z = 0; z < 16; ++z) t += part[z][oi];
        finish(out + o * stride_out, t, alpha, beta);
    }
}

// the matrix-vector view of a problem with m == 1 or n == 1
struct View {
    int64_t outputs, k;
    const void *mat;
    int64_t stride_o, stride_l;
    const void *vec;
    int64_t stride_v;
    int64_t stride_out;
};

View view_of(const Problem &p)
{
    View v{};
    v.k = p.k;
    if (p.n == 1) {
        v.outputs = p.m;
        v.mat = p.A; v.stride_o = p.a_sm(); v.stride_l = p.a_sk();
        v.vec = p.B; v.stride_v = p.b_sk();
        v.stride_out = 1;
    } else {
        v.outputs = p.n;
        v.mat = p.B; v.stride_o = p.b_sn(); v.stride_l = p.b_sk();
        v.vec = p.A; v.stride_v = p.a_sk();
        v.stride_out = p.ldc;
    }
    return v;
}

// R > 0: rows per wavefront of the dot kernel; R = 0: the axpy kernel; R < 0: the panel kernel with LR = -R
template <typename T, int R> struct GemvShape {
    static constexpr bool DOT = R > 0;
    static constexpr int V = 16 / static_cast<int>(sizeof(T));
    static constexpr int OUTPUTS_PER_GROUP = DOT ? 4 * R : (R < 0 ? -R : 64) * V;
    static constexpr int K_GRAIN = DOT ? 64 * V : (R < 0 ? 1024 / (R < 0 ? -R : 1) : 32);          // one round of loads of a work-group
    static int64_t k_per_split(const Problem &p, int split) { return ceil_div(ceil_div(p.k, split), K_GRAIN) * K_GRAIN; }
};

template <typename T, int R> bool gemv_legal(const Problem &p, int split, int64_t)
{
    if ((p.m != 1 && p.n != 1) || p.alpha == 0.f || p.k == 0 || p.fringe_m != 0 || p.fringe_n != 0 || p.clip_m != 0 || p.clip_n != 0) return false;
    if (split < 1 || split > 256 || split > p.k) return false;
    if (p.dtype != (sizeof(T) == 4 ? MG_F32 : MG_F16)) return false;
    const View v = view_of(p);
    if (v.outputs >= (int64_t(1) << 31)) return false;
    // a single output (or a single k) has no stride in that direction: then either kernel applies
    return R > 0 ? (v.stride_l == 1 || v.k == 1) : (v.stride_o == 1 || v.outputs == 1);
}

size_t gemv_workspace(const Problem &p, int split)
{
    return split > 1 ? static_cast<size_t>(split) * static_cast<size_t>(p.m * p.n) * sizeof(float) : 0;
}

template <typename T, int R> hipError_t gemv_launch(const Problem &p, int split)
{
    using S = GemvShape<T, R>;
    const View v = view_of(p);
    float *partial = split > 1 ? static_cast<float *>(p.workspace) : nullptr;
    [[maybe_unused]] const Ends ends = ends_of<T>(v.outputs);
    const dim3 grid(static_cast<unsigned>(ceil_div(v.outputs, S::OUTPUTS_PER_GROUP)), static_cast<unsigned>(split));
    if constexpr (R > 0) {
        hipLaunchKernelGGL((gemv_dot_kernel<T, R>), grid, dim3(256), 0, p.stream, v.outputs, v.k,
                           S::k_per_split(p, split), static_cast<const T *>(v.mat), v.stride_o,
                           static_cast<const T *>(v.vec), v.stride_v, static_cast<T *>(p.C), v.stride_out, partial,
                           p.alpha, p.beta);
    } else if constexpr (R < 0) {
        // A matrix that the last-level cache (256 MB) can still hold from an earlier call or from the kernel that wrote it is read
        // with plain loads, a larger one as a stream: three FP32 matrices in turn, us plain / streamed: 4096^2 (67 MB) 13.0 / 14.2,
        // 4160 x 4096 11.7 / 14.1, 5120^2 (105 MB) 20.0 / 19.8, 8192^2 45.5 / 42.8, 65536 x 2048 91 / 80
        const bool stream = static_cast<double>(v.outputs) * static_cast<double>(v.k) * sizeof(T) > 96.0e6;
        auto flavour = [ends](auto STREAM) {
            constexpr bool streamed = decltype(STREAM)::value;
            return ends == Ends::whole ? gemv_panel_kernel<T, -R, streamed, Ends::whole>
                                       : (ends == Ends::ragged ? gemv_panel_kernel<T, -R, streamed, Ends::ragged> : gemv_panel_kernel<T, -R, streamed, Ends::few>);
        };
        hipLaunchKernelGGL((stream ? flavour(std::true_type{}) : flavour(std::false_type{})), grid, dim3(1024), 0, p.stream, v.outputs, v.k, S::k_per_split(p, split),
                           static_cast<const T *>(v.mat), v.stride_l, static_cast<const T *>(v.vec), v.stride_v,
                           static_cast<T *>(p.C), v.stride_out, partial, p.alpha, p.beta);
    } else {
        hipLaunchKernelGGL((ends == Ends::whole ? gemv_axpy_kernel<T, Ends::whole> : (ends == Ends::ragged ? gemv_axpy_kernel<T, Ends::ragged> : gemv_axpy_kernel<T, Ends::few>)), grid, dim3(256), 0, p.stream, v.outputs, v.k, S::k_per_split(p, split),
                           static_cast<const T *>(v.mat), v.stride_l, static_cast<const T *>(v.vec), v.stride_v,
                           static_cast<T *>(p.C), v.stride_out, partial, p.alpha, p.beta);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || split == 1) return e;
    hipLaunchKernelGGL(gemv_reduce_kernel<T>, dim3(static_cast<unsigned>(ceil_div(v.outputs, 16))), dim3(256), 0,
                       p.stream, partial, split, v.outputs, static_cast<T *>(p.C), v.stride_out, p.alpha, p.beta);
    return hipGetLastError();
}

// tile_m: outputs per work-group; tile_k: elements of the sum one work-group takes per round of loads
template <typename T, int R> KernelEntry gemv_entry(const char *name)
{
    using S = GemvShape<T, R>;
    mg_config c{};
    c.family = MG_FAMILY_GEMV;
    c.dtype = sizeof(T) == 4 ? MG_F32 : MG_F16;
    c.tile_m = S::OUTPUTS_PER_GROUP;
    c.tile_n = 1;
    c.tile_k = S::K_GRAIN;
    c.waves_m = R < 0 ? 16 : 4;
    c.waves_n = 1;
    c.split_k = 1;
    c.threads = R < 0 ? 1024 : 256;
    c.lds_bytes = R > 0 ? 0 : c.waves_m * S::OUTPUTS_PER_GROUP * 4;
    return KernelEntry{name, c, gemv_legal<T, R>, gemv_workspace, gemv_launch<T, R>, nullptr, nullptr};
}

}  // namespace

void register_gemv(std::vector<KernelEntry> &table)
{
    table.push_back(gemv_entry<float, 1>("gemv_dot_f32"));
    table.push_back(gemv_entry<float, 4>("gemv_dot4_f32"));
    table.push_back(gemv_entry<float, 0>("gemv_axpy_f32"));
    table.push_back(gemv_entry<float, -4>("gemv_panel4_f32"));
    table.push_back(gemv_entry<float, -8>("gemv_panel8_f32"));
    table.push_back(gemv_entry<float, -16>("gemv_panel16_f32"));
    table.push_back(gemv_entry<_Float16, 1>("gemv_dot_f16"));
    table.push_back(gemv_entry<_Float16, 4>("gemv_dot4_f16"));
    table.push_back(gemv_entry<_Float16, 0>("gemv_axpy_f16"));
    table.push_back(gemv_entry<_Float16, -4>("gemv_panel4_f16"));
    table.push_back(gemv_entry<_Float16, -8>("gemv_panel8_f16"));
    table.push_back(gemv_entry<_Float16, -16>("gemv_panel16_f16"));
}

}  // namespace mg
