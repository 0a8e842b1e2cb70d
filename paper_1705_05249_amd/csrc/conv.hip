// IM2COL: unfolds one image into the column matrix of its convolution (the IM2COL routine of the paper's
// routine table, Section 3.1; with it a convolution layer becomes the GEMM of Section 1).
//
//   col[(c*KH + kh)*KW + kw][oh*OW + ow] = im[c][oh*stride_h - pad_h + kh*dil_h][ow*stride_w - pad_w + kw*dil_w]
//                                          (0 outside the image), all arrays dense and row-major.
//
// Pure data movement, bound by the write of the column matrix: every thread produces 16 bytes of consecutive
// elements of one matrix row (one vector store per lane, consecutive lanes on consecutive addresses); the image
// is small next to the matrix and is read through the caches.  FP16 with a horizontal stride of one: the 16 bytes are at most two
// runs of consecutive image elements (two output rows, where a row has 16 bytes and more): two 16-byte loads at element alignment
// and a selection, instead of eight loads and their addresses.  us, element by element / runs: 447 channels of 98 x 98, 3 x 3 41.7 /
// 37.9, 48 of 105 x 105, 5 x 5 18.3 / 15.8, 64 of 63 x 63, 7 x 7 16.5 / 15.4; FP32 with its four loads gains nothing (49.6 / 49.6,
// 19.0 / 19.2, 18.2 / 19.0) and stays element by element.
#include "internal.h"

namespace mg {
namespace {

template <typename T, int N> struct __attribute__((packed, aligned(sizeof(T)))) Piece {
    T v[N];
};

// one 16-byte store when the destination allows it, else a store at element alignment
template <typename T, int N> __device__ inline void store(T *dst, const Piece<T, N> &out)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    if (reinterpret_cast<uintptr_t>(dst) % 16 == 0) *reinterpret_cast<u32x4 *>(dst) = __builtin_bit_cast(u32x4, out);
    else *reinterpret_cast<Piece<T, N> *>(dst) = out;
}

// grid.y walks the rows (c, kh, kw) of the column matrix, so everything that depends on the row is wave-uniform
// scalar work; grid.x * 256 threads cover one row, V consecutive columns (oh, ow) per thread.
// RUNS (FP16): stride_w is one and an output row has at least V elements.
template <typename T, bool RUNS>
__global__ __launch_bounds__(256) void im2col_kernel(ConvShape s, uint32_t out_h, uint32_t out_w, uint32_t rows,
                                                      const T *__restrict__ im, T *__restrict__ col)
{
    constexpr int V = 16 / static_cast<int>(sizeof(T));
    const uint32_t per_row = out_h * out_w;
    const uint32_t j0 = (blockIdx.x * 256u + threadIdx.x) * V;
    if (j0 >= per_row) return;
    const uint32_t count = per_row - j0 < V ? per_row - j0 : V;
    const uint32_t kw_n = static_cast<uint32_t>(s.kernel_w), kh_n = static_cast<uint32_t>(s.kernel_h);
    const int height = static_cast<int>(s.height), width = static_cast<int>(s.width);
    const int stride_h = static_cast<int>(s.stride_h), stride_w = static_cast<int>(s.stride_w);
    const uint32_t oh0 = j0 / out_w, ow0 = j0 % out_w;
    [[maybe_unused]] const int64_t total = s.channels * s.height * s.width;
    for (uint32_t r = blockIdx.y; r < rows; r += gridDim.y) {
        const uint32_t kw = r % kw_n, kh = (r / kw_n) % kh_n, c = r / (kw_n * kh_n);
        const int ih0 = static_cast<int>(kh) * static_cast<int>(s.dilation_h) - static_cast<int>(s.pad_h);
        const int iw0 = static_cast<int>(kw) * static_cast<int>(s.dilation_w) - static_cast<int>(s.pad_w);
        const T *plane = im + static_cast<int64_t>(c) * height * width;
        if constexpr (RUNS) {
            // elements 0 .. first - 1 lie in output row oh0, the others in the next; the second run is loaded from where its
            // element 0 would lie.  Both may start before the image or end behind it (padding): such threads go element by element
            int first = static_cast<int>(out_w - ow0 < V ? out_w - ow0 : V);
            asm volatile("" : "+v"(first));        // (known to be above 0, the second run is loaded in pieces, less its element 0)
            const int ih = static_cast<int>(oh0) * stride_h + ih0, iw = static_cast<int>(ow0) + iw0;
            const int64_t in_plane = static_cast<int64_t>(ih) * width + iw;
            const int64_t run0 = static_cast<int64_t>(c) * height * width + in_plane;
            const int64_t run1 = run0 + static_cast<int64_t>(stride_h) * width - static_cast<int>(out_w);
            if (count == V && run0 >= 0 && run1 >= 0 && run0 + V <= total && (first == V || run1 + V <= total)) {
                const Piece<T, V> a = *reinterpret_cast<const Piece<T, V> *>(im + run0);
                const Piece<T, V> b = *reinterpret_cast<const Piece<T, V> *>(im + (first == V ? run0 : run1));
                const bool row0 = ih >= 0 && ih < height, row1 = ih + stride_h >= 0 && ih + stride_h < height;
                Piece<T, V> out;
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const bool second = e >= first;
                    const int x = iw + e - (second ? static_cast<int>(out_w) : 0);
                    const bool in = (second ? row1 : row0) && x >= 0 && x < width;
                    out.v[e] = in ? (second ? b.v[e] : a.v[e]) : static_cast<T>(0.f);
                }
                store(col + static_cast<int64_t>(r) * per_row + j0, out);
                continue;
            }
        }
        // first every address (0 stands in where the element is padding or past the row's end), then all
        // loads at once, so that the loads of one thread overlap instead of waiting for each other
        int at[V];
        bool inside[V];
        uint32_t oh = oh0, ow = ow0;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const int ih = static_cast<int>(oh) * stride_h + ih0, iw = static_cast<int>(ow) * stride_w + iw0;
            inside[e] = static_cast<uint32_t>(e) < count && ih >= 0 && ih < height && iw >= 0 && iw < width;
            at[e] = inside[e] ? ih * width + iw : 0;
            if (++ow == out_w) {
                ow = 0;
                ++oh;
            }
        }
        Piece<T, V> out;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const T x = plane[at[e]];
            out.v[e] = inside[e] ? x : static_cast<T>(0.f);
        }
        T *dst = col + static_cast<int64_t>(r) * per_row + j0;
        if (count == V) {
            store(dst, out);
        } else {
            // (unrolled with constant indices: a run-time index would move `out` out of registers)
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (static_cast<uint32_t>(e) < count) dst[e] = out.v[e];
        }
    }
}

}  // namespace

int64_t conv_out_extent(int64_t size, int64_t kernel, int64_t pad, int64_t stride, int64_t dilation)
{
    const int64_t span = size + 2 * pad - dilation * (kernel - 1) - 1;
    return span < 0 ? 0 : span / stride + 1;
}

hipError_t launch_im2col(int dtype, const ConvShape &s, const void *im, void *col, hipStream_t stream)
{
    const int64_t out_h = conv_out_extent(s.height, s.kernel_h, s.pad_h, s.stride_h, s.dilation_h);
    const int64_t out_w = conv_out_extent(s.width, s.kernel_w, s.pad_w, s.stride_w, s.dilation_w);
    const int64_t rows = s.channels * s.kernel_h * s.kernel_w;     // rows * out_h * out_w < 2^31, checked by the caller
    if (rows * out_h * out_w == 0) return hipSuccess;
    const int per_thread = dtype == MG_F32 ? 4 : 8;
    const dim3 grid(static_cast<unsigned>(ceil_div(out_h * out_w, 256 * per_thread)),
                    static_cast<unsigned>(rows < 65535 ? rows : 65535));
    const bool runs = s.stride_w == 1 && out_w >= per_thread;
    auto launch = [&](auto kernel, auto element) {
        using T = decltype(element);
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, s, static_cast<uint32_t>(out_h), static_cast<uint32_t>(out_w),
                           static_cast<uint32_t>(rows), static_cast<const T *>(im), static_cast<T *>(col));
    };
    if (dtype == MG_F32) launch(im2col_kernel<float, false>, 0.f);
    else runs ? launch(im2col_kernel<_Float16, true>, _Float16(0)) : launch(im2col_kernel<_Float16, false>, _Float16(0));
    return hipGetLastError();
}

}  // namespace mg
