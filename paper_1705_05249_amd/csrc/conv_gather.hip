// Convolution of one image in one launch, for layers of few outputs: the column matrix of IM2COL (paper, Section 3.1) is never stored, nor
// gathered from memory element by element.  A work-group owns 32 output positions x 32 filters; what the 32 positions see of the
// image, a band of a few rows of every channel, is copied into LDS with its zero padding around it, so that a tap of any output is an
// address (that of the position plus that of the row (c, kh, kw) of the column matrix, from a table) without conditions.  The eight
// wavefronts share the sum: each takes an eighth of the rows of the column matrix, reads its MFMA operand from the band element by element and
// the filters' one straight from memory (16 bytes per lane, contiguous along the sum), and the eight partial blocks meet in LDS (as in tiny.hip).
//
// Bound by latency: launch, the rounds of loads that bring the band (0.9 us each: PIECES pieces of a thread) and the LDS reads of an eighth of
// the sum (0.32 us per K-step).  The unfold route takes two dependent launches, each with a gap of 3.5-4 us and a latency of its own.  us,
// unfold route / this kernel: FP16 128 channels of 28 x 28, 3 x 3, 256 filters 11.8 / 7.6, 256 of 14 x 14, 512 filters 21.0 / 11.7, 128 of 56 x
// 56, 128 filters 16.2 / 11.7; FP32 the first 19.1 / 11.7; 16 of 7 x 7, 16 filters 8.9 / 4.3 (FP32 7.7 / 4.7).
// Tried: sixteen wavefronts (the first layer 8.7, the fourth 5.0), ten K-steps of filters at once (7.8, 4.6), K-steps in groups of three without
// branches (7.7, 5.6), 16 x 16 blocks, whose filter loads are 64-byte runs (7.6, 4.8).
#include "mfma_host.h"

namespace mg {
namespace {

struct GatherArgs {
    const void *im, *weights;
    void *out;
    ConvGeom g;
    int positions, filters, k;
    int chunk;                     // channels of the image band that are in LDS at once
    int pitch, left;               // elements of a row of the band; of them in front of the image's first column
    int band_bytes;                // LDS bytes of the band (the table lies behind it)
    uint32_t by_taps, by_kw, by_row, by_ow;       // for divisions by kh * kw, kw, pieces of an image row, ow
    int line_step;                 // image rows that a thread's pieces are apart
    int share, rest, minor, positions_first;      // as in TinyArgs
    float alpha, beta;
};

constexpr int kThreads = 512;

// n / d by the multiplication with ceil(2^32 / d), exact while n * d < 2^32; 0 stands for d == 1
uint32_t reciprocal(int64_t d) { return d == 1 ? 0u : static_cast<uint32_t>(((int64_t(1) << 32) + d - 1) / d); }
__device__ inline int quotient(int n, uint32_t by) { return by == 0 ? n : static_cast<int>(__umulhi(static_cast<uint32_t>(n), by)); }

constexpr int kReduceBytes = 8 * 16 * 64 * 4 + 32 * 33 * 4;     // partial blocks and the staged sums

// V: elements of a piece of an image row (a divisor of its length, at most 16 bytes)
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void conv_gather_kernel(const GatherArgs a)
{
    constexpr int CH = ElemTraits<T>::CH, STEP = 2 * CH;       // values of k per lane and per K-step
    // K-steps whose filters are loaded together (FP32: six in place of four took 120 layers 2.5 % longer in the mean)
    constexpr int BATCH = sizeof(T) == 4 ? 4 : 6;
    constexpr int PIECES = 8;                                   // pieces of the band a thread has in flight
    constexpr int ES = sizeof(T);
    using Raw = std::conditional_t<V * ES == 16, u32x4, std::conditional_t<V * ES == 8, u32x2, std::conditional_t<V * ES == 4, uint32_t, uint16_t>>>;
    struct __attribute__((packed, aligned(ES))) Loose { T v[V]; };          // at element alignment
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const ConvGeom &g = a.g;
    const int tid = threadIdx.x, lane = tid % 64, ln = lane % 32, lg = lane / 32;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);

    const int xcd = blockIdx.x % 8;
    const int id = xcd * a.share + (xcd < a.rest ? xcd : a.rest) + blockIdx.x / 8;
    const int outer = id / a.minor, inner = id - outer * a.minor;
    const int m0 = (a.positions_first ? inner : outer) * 32, n0 = (a.positions_first ? outer : inner) * 32;
    const T *__restrict__ im = static_cast<const T *>(a.im);
    const T *__restrict__ weights = static_cast<const T *>(a.weights);

    // the band: rows of the image from first_row on, band_rows of each channel
    const int last = m0 + 31 < a.positions ? m0 + 31 : a.positions - 1;
    const int oh_first = quotient(m0, a.by_ow);
    const int band_rows = (quotient(last, a.by_ow) - oh_first) * g.stride_h + (g.kh - 1) * g.dil_h + 1;
    const int first_row = oh_first * g.stride_h - g.pad_h;
    const int taps = g.kh * g.kw;
    const int per_row = g.w / V;                                // pieces of an image row (V: a power of two)
    int *const table = reinterpret_cast<int *>(lds + a.band_bytes);

    // this lane's position in the band (lanes past the last output repeat it; they are not stored)
    const int pos = m0 + ln < a.positions ? m0 + ln : a.positions - 1;
    const int oh = quotient(pos, a.by_ow), ow = pos - oh * g.ow;
    const char *const mine = lds + (((oh - oh_first) * g.stride_h) * a.pitch + ow * g.stride_w - g.pad_w + a.left) * ES;
    const int filter = n0 + ln < a.filters ? n0 + ln : a.filters - 1;
    const T *const w_row = weights + static_cast<int64_t>(filter) * a.k;

    // old values of this thread's two outputs (position tid % 32, filters tid / 32 and + 16): asked for now
    T *out = static_cast<T *>(a.out);
    bool stored[2];
    float old[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int mi = tid % 32, ni = tid / 32 + 16 * i;
        stored[i] = m0 + mi < a.positions && n0 + ni < a.filters;
        if (stored[i] && a.beta != 0.f) old[i] = load_as_float(out + (m0 + mi) + static_cast<int64_t>(n0 + ni) * a.positions);
    }
    // FP32: two sets, for even and odd values of k of a lane's four, added at the end.  One set makes a sum eight chains of k / 8 terms; the unfold
    // route cuts long sums into up to sixteen slices.  Error against 64 bits, that route / one set / two / four: k = 1377 2.1e-7 / 2.4e-7 / 1.8e-7 / 1.4e-7, 3546
    // 2.7e-7 / 3.8e-7 / 2.7e-7 / 2.0e-7.  Two hold it over 410 layers where the route sums on the FP32 pipes; four take 14 registers more than let two
    // work-groups share a compute unit, or shorter batches, with which long sums are up to 26 % slower.
    constexpr int SETS = ES == 4 ? 2 : 1;
    floatx16 acc[SETS] = {};
    auto multiply = [&](const u32x4 &filters, const u32x4 &positions) __attribute__((always_inline)) {
        if constexpr (ES == 2) {
            mma(acc[0], filters, positions, T{});
        } else {
            // (whole-vector casts and named components, see mma)
            const floatx4 p = __builtin_bit_cast(floatx4, positions), f = __builtin_bit_cast(floatx4, filters);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(p.x, f.x, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(p.y, f.y, acc[1], 0, 0, 0);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(p.z, f.z, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(p.w, f.w, acc[1], 0, 0, 0);
        }
    };

    // the padding around the image stays zero in every chunk: cleared once
    for (int at = tid * 16; at < a.band_bytes; at += kThreads * 16) *reinterpret_cast<u32x4 *>(lds + at) = u32x4{0u, 0u, 0u, 0u};
    // addresses of the column matrix's rows relative to a position's, for a chunk's channels (the last chunk may have fewer)
    for (int r = tid; r < ((a.chunk * taps + STEP - 1) / STEP) * STEP; r += kThreads) {
        const int c = quotient(r, a.by_taps), t = r - c * taps, kh = quotient(t, a.by_kw), kw = t - kh * g.kw;
        table[r] = r < a.chunk * taps ? ((c * band_rows + kh * g.dil_h) * a.pitch + kw * g.dil_w) * ES : 0;
    }
    __syncthreads();

    // a thread's pieces are line_step lines (rows of the band) and piece_step pieces apart
    const float by_band = 1.f / static_cast<float>(band_rows);             // (halves added: exact for the numbers of lines there are)
    const int line_step = a.line_step, piece_step = kThreads - line_step * per_row;
    const int channel_step = static_cast<int>((static_cast<float>(line_step) + 0.5f) * by_band), row_step = line_step - channel_step * band_rows;
    const int line0 = quotient(tid, a.by_row), piece0 = tid - line0 * per_row;
    const int channel0 = static_cast<int>((static_cast<float>(line0) + 0.5f) * by_band);
    for (int c0 = 0; c0 < g.channels; c0 += a.chunk) {
        const int channels = g.channels - c0 < a.chunk ? g.channels - c0 : a.chunk;
        const int k0 = c0 * taps, kc = channels * taps;         // rows of the column matrix in this chunk
        // whole K-steps, in shares that differ by one at most: with all but the last rounded up, the chains of an FP32 sum of 72 to 147 terms
        // are longer on fewer wavefronts and its error is 2 to 4 % larger.  What is left behind them is the first wavefront's, whose
        // share is of the smaller ones.
        const int steps = kc / STEP;
        const int s_begin = steps * wave / 8, s_end = steps * (wave + 1) / 8;
        const T *const w_mine = w_row + k0 + lg * CH;
        // filters of K-steps s .. s + BATCH - 1 (past the end: the last one again)
        auto load_filters = [&](u32x4 (&q)[BATCH], int s) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < BATCH; ++j) q[j] = load_unaligned_chunk<T>(w_mine + (s + j < s_end ? s + j : s_end - 1) * STEP);
        };
        u32x4 now[BATCH] = {}, next[BATCH] = {};
        if (s_begin < s_end) load_filters(now, s_begin);

        // the band: every piece of a row of the image inside it; a thread walks pieces kThreads apart
        const int pieces = channels * band_rows * per_row;
        int piece = piece0, channel = channel0, row = line0 - channel0 * band_rows;
        for (int base = 0; base < pieces; base += PIECES * kThreads) {
            Raw v[PIECES];
            int to[PIECES];
            static_for<PIECES>([&](auto P) __attribute__((always_inline)) {
                constexpr int p = decltype(P)::value;
                const int ih = first_row + row;
                const bool in = channel < channels && static_cast<unsigned>(ih) < static_cast<unsigned>(g.h);
                to[p] = in ? ((channel * band_rows + row) * a.pitch + a.left + piece * V) * ES : -1;
                // (a piece that is not wanted: the image's first one)
                v[p] = __builtin_bit_cast(Raw, *reinterpret_cast<const Loose *>(im + (in ? (static_cast<int64_t>(c0 + channel) * g.h + ih) * g.w + piece * V : 0)));
                piece += piece_step;
                row += row_step;
                channel += channel_step;
                if (piece >= per_row) { piece -= per_row; ++row; }
                if (row >= band_rows) { row -= band_rows; ++channel; }
            });
            static_for<PIECES>([&](auto P) __attribute__((always_inline)) {
                constexpr int p = decltype(P)::value;
                if (to[p] >= 0) *reinterpret_cast<Raw *>(lds + to[p]) = v[p];
            });
        }
        __syncthreads();

        // the positions' operand of K-step s; wanted: rows of the column matrix that exist from the lane's first one on
        auto gather = [&](int s, int wanted) __attribute__((always_inline)) {
            const int *t = table + s * STEP + lg * CH;
            u32x4 fa = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < CH; ++e) {
                const uint32_t x = elem_bits<T>(*reinterpret_cast<const T *>(mine + t[e]));
                const uint32_t b = e < wanted ? x : 0u;
                if constexpr (ES == 4) fa[e] = b;
                else fa[e >> 1] |= b << (16 * (e & 1));
            }
            return fa;
        };
        for (int s = s_begin; s < s_end; s += BATCH) {
            if (s + BATCH < s_end) load_filters(next, s + BATCH);
            static_for<BATCH>([&](auto J) __attribute__((always_inline)) {
                constexpr int j = decltype(J)::value;
                if (s + j < s_end) multiply(now[j], gather(s + j, CH));
            });
#pragma unroll
            for (int j = 0; j < BATCH; ++j) now[j] = next[j];
        }
        if (wave == 0 && steps * STEP < kc) {
            const int left = kc - steps * STEP - lg * CH;
            multiply(gather_chunk<T>(w_mine + steps * STEP, left), gather(steps, left));
        }
        __syncthreads();               // everyone is done with the band
    }

    // the eight partial blocks, as in tiny_gemm_kernel
    float *part = reinterpret_cast<float *>(lds);
    float *stage = reinterpret_cast<float *>(lds + 8 * 16 * 64 * 4);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        float sum = acc[0][r];
        if constexpr (SETS == 2) sum += acc[1][r];
        part[(wave * 16 + r) * 64 + lane] = sum;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = tid + kThreads * i, r = e / 64, l = e % 64;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) s += part[w * 1024 + e];
        stage[(l % 32) * 33 + 8 * (r / 4) + 4 * (l / 32) + r % 4] = s;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int mi = tid % 32, ni = tid / 32 + 16 * i;
        if (stored[i]) {
            float o = a.alpha * stage[ni * 33 + mi];
            if (a.beta != 0.f) o = fmaf(a.beta, old[i], o);
            store_from_float(out + (m0 + mi) + static_cast<int64_t>(n0 + ni) * a.positions, o);
        }
    }
}

template <typename T, int V> hipError_t launch(const GatherArgs &a, int lds_bytes, hipStream_t stream)
{
    auto kernel = conv_gather_kernel<T, V>;
    static bool attr_set = false;   // raising the dynamic LDS limit is idempotent; races are harmless
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const unsigned groups = static_cast<unsigned>(ceil_div(a.positions, 32) * ceil_div(a.filters, 32));
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(kThreads), lds_bytes, stream, a);
    return hipGetLastError();
}

struct Band {
    int v, left, pitch;
    int64_t rows, chunk, band_bytes, lds_bytes;
};

// The band of a layer: chunk 0 if not even sixteen channels of it (or all, if fewer) fit into LDS
Band band_of(int dtype, const ConvShape &s, int64_t out_h, int64_t out_w)
{
    const int64_t es = dtype == MG_F32 ? 4 : 2, taps = s.kernel_h * s.kernel_w;
    Band b{};
    b.v = static_cast<int>(16 / es);
    while (s.width % b.v != 0) b.v /= 2;
    b.left = static_cast<int>(ceil_div(s.pad_w, b.v) * b.v);
    b.pitch = static_cast<int>(ceil_div(b.left + s.width + s.pad_w, b.v) * b.v);
    int64_t lines = (31 + out_w - 1) / out_w;               // output rows that 32 positions span, less one
    if (lines > out_h - 1) lines = out_h - 1;
    b.rows = lines * s.stride_h + (s.kernel_h - 1) * s.dilation_h + 1;
    const int64_t room = 144 * 1024, step = 2 * (16 / es);
    auto bytes = [&](int64_t channels) {
        b.band_bytes = ceil_div(channels * b.rows * b.pitch * es, 16) * 16;
        return b.band_bytes + ceil_div(channels * taps, step) * step * 4;
    };
    b.chunk = s.channels;
    while (b.chunk > 16 && bytes(b.chunk) > room) b.chunk = ceil_div(b.chunk / 2, 16) * 16 < b.chunk ? ceil_div(b.chunk / 2, 16) * 16 : 16;
    b.lds_bytes = bytes(b.chunk);
    if (b.lds_bytes > room) b.chunk = 0;
    if (b.lds_bytes < kReduceBytes) b.lds_bytes = kReduceBytes;
    return b;
}

}  // namespace

bool conv_gather_fits(int dtype, const ConvShape &s, int64_t filters)
{
    const int64_t out_h = conv_out_extent(s.height, s.kernel_h, s.pad_h, s.stride_h, s.dilation_h);
    const int64_t out_w = conv_out_extent(s.width, s.kernel_w, s.pad_w, s.stride_w, s.dilation_w);
    const int64_t lim = int64_t(1) << 31;
    // (the extents of the band are worked out in 32 bits)
    if (s.pad_w > 4096 || s.width > 65536 || (s.kernel_h - 1) * s.dilation_h > 65536 || s.stride_h > 4096 || s.kernel_h * s.kernel_w > 4096) return false;
    if (s.channels * s.kernel_h * s.kernel_w >= lim || out_h * out_w >= lim - 32 || filters >= lim - 32) return false;
    if (ceil_div(out_h * out_w, 32) * ceil_div(filters, 32) >= lim) return false;
    // (divisions by multiplication: the dividends are positions, rows of the column matrix in LDS and threads)
    if ((out_h * out_w + 32) * out_w >= (int64_t(1) << 32) || s.kernel_h * s.kernel_w * 65536 >= (int64_t(1) << 32)) return false;
    return band_of(dtype, s, out_h, out_w).chunk != 0;
}

// The route of a layer: this kernel, the GEMM kernel that gathers the column matrix from memory (up to 256 terms and 64 filters), or the unfold pass and a
// GEMM.  All estimates in us, fitted to each route forced in one build on 18000 (FP16) and 17000 (FP32) random layers: 1 to 512 channels, 4 to 300 wide, filters of 1 x 1
// to 7 x 7, strides, paddings and dilations up to 3 and 4, 1 to 512 filters; rms errors: here 6 and 4.5 %, gathering GEMM 7 and 6, unfold 7 and 6.5.  A gain of 3 % is asked for, of
// 12 % with several turns or chunks, whose estimates are further off; past eight turns it did not pay.  Here: rounds of loads that bring the band and the LDS reads of the
// sum make a work-group's latency, of which a second work-group on a compute unit hides all but its loads and K-steps; what the grid reads counts beside that.
// On 16000 other layers calls take 0.67 of the time without this kernel, 41 are more than 3 % slower (at most 1.27 times).  By the rule before (one sum of six terms for
// the other routes, a gain of 1.4 for FP32 layers of several chunks or turns) 65 of 7300 were, up to 1.38 times; against that rule without the 1.4, 0.93 of the time and
// 188 of 16000 more than 3 % slower.  us, unfold or gathering GEMM / this: FP32 64 channels of 140 x 140, 3 x 3, 22 filters 40.7 / 25.2, 480 of 64 x 64, 5 x 5, stride 2, 249 filters 80 / 96, 219 of
// 185 x 6, 7 x 3, 14 filters 689 / 29 (a thin product); FP16 7 of 116 x 116, 3 x 3, 32 filters 6.1 / 8.5, 447 of 98 x 98, 3 x 3, 32 filters 62 / 114.
ConvRoute conv_route(int dtype, const ConvShape &s, int64_t filters)
{
    const bool f32 = dtype == MG_F32;
    const int64_t out_h = conv_out_extent(s.height, s.kernel_h, s.pad_h, s.stride_h, s.dilation_h);
    const int64_t out_w = conv_out_extent(s.width, s.kernel_w, s.pad_w, s.stride_w, s.dilation_w);
    const int64_t taps = s.kernel_h * s.kernel_w, terms = s.channels * taps, positions = out_h * out_w, es = f32 ? 4 : 2;
    const int64_t groups = ceil_div(positions, 32) * ceil_div(filters, 32), thinner = positions < filters ? positions : filters;
    const double k = static_cast<double>(terms), x = static_cast<double>(groups) / 256.0;
    const double tiles = static_cast<double>(ceil_div(positions, 64)) * static_cast<double>(ceil_div(filters, 64)) / 256.0;       // of 64 x 64, for a compute unit
    const double busy = tiles < 1.0 ? tiles : 1.0, over = tiles > 1.0 ? tiles - 1.0 : 0.0, ktiles = static_cast<double>(ceil_div(terms, f32 ? 32 : 64));
    const double column_mb = 1.0e-6 * k * static_cast<double>(positions) * static_cast<double>(es);
    const double image_mb = 1.0e-6 * static_cast<double>(s.channels) * static_cast<double>(s.height * s.width) * static_cast<double>(es);
    const double gflop = 2.0e-9 * k * static_cast<double>(positions) * static_cast<double>(filters);
    // (FP16: rows of the product's operands, filters and column matrix, off 16 bytes)
    const double off_f = !f32 && terms % 8 != 0 ? 1.0 : 0.0, off_c = !f32 && positions % 8 != 0 ? 1.0 : 0.0, off = off_f + off_c > 0.0 ? 1.0 : 0.0;

    // the unfold pass and a matrix-vector product, the kernel whose wavefronts share a sum, the one for thin products, or tiles
    double unfold;
    const int64_t most_shared = f32 ? (groups > 64 ? 1536 : 1280) + (thinner < 16 ? (groups > 64 ? 512 : 256) : 0) : 2560;
    const double pass = f32 ? (positions % 8 != 0 ? 0.473 : 0.428) * column_mb + 0.030 * image_mb : (0.511 + 0.098 * off_c) * column_mb + 0.061 * image_mb;
    if (thinner == 1) {
        unfold = pass + (f32 ? 5.13 + 0.099 * column_mb + 0.00158 * k : 6.19 + 0.218 * column_mb + 0.00189 * k);
    } else if (groups <= 256 && terms >= 48 && terms <= most_shared) {
        unfold = f32 ? pass + 5.57 + 0.00701 * k + 0.937 * x
                     : 6.01 + 0.778 * column_mb + 0.022 * image_mb + (0.00267 + 0.00045 * off_c) * k + 0.878 * off_f + 0.506 * off_c;
    } else if (thinner < 16) {
        unfold = pass + (f32 ? 5.51 + 0.132 * k + 0.32 * column_mb : 5.93 + 0.143 * k + 0.70 * column_mb);
    } else {
        const double wide = ktiles * (tiles > 0.05 ? tiles : 0.05);
        const double sliced = f32 ? 4.31 + 2.44 * sqrt(wide) : 4.69 + 1.59 * sqrt(wide), whole = (f32 ? 0.580 : 0.421) * ktiles, sum = sliced < whole ? sliced : whole;
        unfold = f32 ? pass + 6.88 + sum + 1.17 * over + 4.05 * gflop + 0.227 * x
                     : 6.10 + 0.534 * column_mb + 0.063 * image_mb + sum * (1.0 + 0.111 * (off_f + off_c)) + 0.392 * over + (0.042 + 1.07 * off) * gflop + 0.120 * x +
                           0.597 * off_f + 0.877 * off_c;
    }
    ConvRoute route = ConvRoute::unfold;
    double best = unfold;
    if (terms <= 256 && filters <= 64) {
        const double late = tiles > 0.753 ? tiles - 0.753 : 0.0;
        const double fused = f32 ? 4.61 + 1.277 * ktiles + 1.248 * late * (1.0 + 0.657 * ktiles) + 0.203 * ktiles * busy
                                 : 4.38 + 1.608 * ktiles + 1.119 * late * (1.0 + 0.439 * ktiles) + 0.098 * ktiles * busy + 0.060 * column_mb;
        if (1.03 * fused < best) {
            route = ConvRoute::fused;
            best = fused;
        }
    }
    if (groups > 8 * 256 || !conv_gather_fits(dtype, s, filters)) return route;
    const Band b = band_of(dtype, s, out_h, out_w);
    // rows of the band of most work-groups (b.rows is the most that any can have)
    int64_t lines = out_w % 32 == 0 ? 0 : (32 % out_w == 0 ? 32 / out_w - 1 : (30 + out_w) / out_w);
    if (lines > out_h - 1) lines = out_h - 1;
    int64_t rows = lines * s.stride_h + (s.kernel_h - 1) * s.dilation_h + 1;
    if (rows > s.height) rows = s.height;
    const int64_t step = f32 ? 8 : 16;
    const int64_t chunks = ceil_div(s.channels, b.chunk), last = s.channels - (chunks - 1) * b.chunk, per_channel = rows * (s.width / b.v);
    const double rounds = static_cast<double>(ceil_div(b.chunk * per_channel, 8 * kThreads) * (chunks - 1) + ceil_div(last * per_channel, 8 * kThreads));
    const double loads = static_cast<double>(ceil_div(b.chunk * per_channel, kThreads) * (chunks - 1) + ceil_div(last * per_channel, kThreads));
    const double steps = static_cast<double>(ceil_div(b.chunk * taps / step, 8) * (chunks - 1) + ceil_div(last * taps / step, 8));
    const double partial = static_cast<double>((b.chunk * taps % step != 0 ? chunks - 1 : 0) + (last * taps % step != 0 ? 1 : 0));
    // loads of filters by a wavefront, whole batches of six K-steps on as many wavefronts as have any: from rows at odd elements each takes its time
    auto batches = [&](int64_t channels) {
        const int64_t all = channels * taps / step;
        return static_cast<double>((all < 8 ? all : 8) * ceil_div(ceil_div(all, 8), 6)) * (6.0 / 8.0);
    };
    const double fill = static_cast<double>(filters < 32 ? filters : 32) / 32.0;        // distinct rows of filters
    const double odd = !f32 && terms % 2 != 0 ? fill * (batches(b.chunk) * static_cast<double>(chunks - 1) + batches(last)) : 0.0;
    const double latency = (f32 ? 0.748 : 0.783) + (f32 ? 0.778 : 0.726) * rounds + (f32 ? 0.0332 : 0.0466) * loads + (f32 ? 2.20 : 0.917) * k / kThreads + 0.353 * odd +
                           (f32 ? 0.42 : 0.37) * static_cast<double>(chunks - 1) + (f32 ? 0.045 : 0.0) * steps + (f32 ? 0.458 : 0.350) * static_cast<double>(b.lds_bytes) / 65536.0;
    const double another = (f32 ? 0.891 : 0.966) + (f32 ? 0.0085 : 0.0368) * loads + (f32 ? 0.277 : 0.057) * (steps + partial) + 0.243 * odd;
    const int64_t resident = b.lds_bytes <= 80 * 1024 ? 2 : 1, full = groups / (resident * 256), rest = groups % (resident * 256);
    const double reads_kb = (static_cast<double>(s.channels * rows * s.width) + static_cast<double>(filters < 32 ? filters : 32) * k) * static_cast<double>(es) / 1024.0;
    const double here = (f32 ? 2.58 : 2.71) + static_cast<double>(full) * (latency + static_cast<double>(resident - 1) * another) +
                        (rest > 0 ? latency + (rest > 256 ? another : 0.0) : 0.0) + (f32 ? 0.0066 : 0.0103) * x * reads_kb;
    // (FP32: the gathering GEMM kernel adds its terms in one chain, with 1.45 times the error of eight at 27 terms: only for a clear gain)
    const bool several = groups > 256 || chunks > 1;
    const double asked = f32 && route == ConvRoute::fused ? (several ? 1.08 : 0.9) : (several ? 1.12 : 1.03);
    return asked * here < best ? ConvRoute::gather : route;
}

hipError_t launch_conv_gather(int dtype, const ConvShape &s, int64_t filters, float alpha, const void *im, const void *weights, float beta,
                              void *out, hipStream_t stream)
{
    GatherArgs a{};
    a.im = im; a.weights = weights; a.out = out;
    a.g = conv_geometry(s);
    a.positions = a.g.oh * a.g.ow;
    a.filters = static_cast<int>(filters);
    a.k = static_cast<int>(s.channels * s.kernel_h * s.kernel_w);
    const Band b = band_of(dtype, s, a.g.oh, a.g.ow);
    if (b.chunk == 0) return hipErrorInvalidValue;
    a.chunk = static_cast<int>(b.chunk);
    a.pitch = b.pitch;
    a.left = b.left;
    a.band_bytes = static_cast<int>(b.band_bytes);
    a.alpha = alpha; a.beta = beta;
    a.by_taps = reciprocal(s.kernel_h * s.kernel_w);
    a.by_kw = reciprocal(s.kernel_w);
    a.by_row = reciprocal(s.width / b.v);
    a.by_ow = reciprocal(a.g.ow);
    a.line_step = static_cast<int>(kThreads / (s.width / b.v));
    const int64_t across_m = ceil_div(a.positions, 32), across_n = ceil_div(filters, 32), groups = across_m * across_n;
    a.share = static_cast<int>(groups / 8);
    a.rest = static_cast<int>(groups % 8);
    a.positions_first = across_m <= across_n ? 1 : 0;
    a.minor = static_cast<int>(a.positions_first ? across_m : across_n);
    const int lds = static_cast<int>(b.lds_bytes);
    if (dtype == MG_F32) {
        if (b.v == 4) return launch<float, 4>(a, lds, stream);
        return b.v == 2 ? launch<float, 2>(a, lds, stream) : launch<float, 1>(a, lds, stream);
    }
    if (b.v == 8) return launch<_Float16, 8>(a, lds, stream);
    if (b.v == 4) return launch<_Float16, 4>(a, lds, stream);
    return b.v == 2 ? launch<_Float16, 2>(a, lds, stream) : launch<_Float16, 1>(a, lds, stream);
}

}  // namespace mg
