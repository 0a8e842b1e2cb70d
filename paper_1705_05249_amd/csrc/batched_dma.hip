// Strided batches of FP16 instances whose rows start on 16 bytes: the direct-to-LDS tiles for sizes that end anywhere (mfma_dma_kernel.h), a grid of
// the tiles of all instances.  (Only strided batches: the offsets of the others are on the device, their alignment is not known.)
// Bound by latency for calls that the chip holds at once (launch, one load, the products of a K-tile or two, the turn through LDS and one store:
// 512 x (128, 128, 64) in 8.6 us of which the traffic of its 33 MB takes 5), else by traffic.  The kernel of batched_tile.hip brings 64 x 64
// tiles through registers, so that a 128 x 128 instance asks for its operands twice and takes four work-groups.  us in a replayed graph (A along m, B along
// k), that kernel / this one: 512 x (128, 128, 64) 11.5 / 8.6, 4000 of them (262 MB, not taken) 52 / 53, 500 x 128^3 13.0 / 10.5, 1000 x 96^3 18.4 / 15.4, 200 x 160^3
// 13.4 / 10.7, 200 x (64, 72, 136) 6.9 / 4.7, 3000 x 48^3 12.5 / 11.5.  Two LDS stages; three take a compute unit's second work-group (1.3 times as long).
#include "batched_walk.h"
#include "mfma_dma_kernel.h"
#include "mfma_host.h"

namespace mg {
namespace {

struct BatchArgs {
    batchwalk::Divisor tiles;              // of an instance
    int64_t stride_a, stride_b, stride_c;
};

template <int BM, int BN, int WM, int WN, bool AK, bool BKC, int STAGES>
__global__ __launch_bounds__(WM *WN * 64) void hbatched_dma_kernel(const MfmaArgs args, const BatchArgs batch)
{
#if defined(__HIP_DEVICE_COMPILE__)
    // the tiles of an instance one after the other on one XCD: they share its operands in the XCD's L2
    const int total = gridDim.x, xcd = blockIdx.x % 8, q = total / 8, rem = total % 8;
    const uint32_t id = static_cast<uint32_t>(xcd * q + (xcd < rem ? xcd : rem) + blockIdx.x / 8);
    const uint32_t instance = batch.tiles.quot(id);
    const int tile = static_cast<int>(id - instance * batch.tiles.d);
    MfmaArgs mine = args;
    mine.A = static_cast<const _Float16 *>(args.A) + instance * batch.stride_a;
    mine.B = static_cast<const _Float16 *>(args.B) + instance * batch.stride_b;
    mine.C = static_cast<_Float16 *>(args.C) + instance * batch.stride_c;
    mine.partial = nullptr;
    mine.mask = 0;
    const int tn = tile / args.tiles_m, tm = tile - tn * args.tiles_m;
    hgemm_dma_tile<BM, BN, WM, WN, AK, BKC, 16, DMA_RAGGED, false, STAGES>(mine, static_cast<int64_t>(tm) * BM, static_cast<int64_t>(tn) * BN, 0, args.k);
#else
    (void)args;
    (void)batch;
#endif
}

template <int BM, int BN, int WM, int WN, bool AK, bool BKC, int STAGES> hipError_t launch(const BatchedProblem &p)
{
    constexpr int EPILOGUE = WM * WN * 32 * ((BM / WM) * 4 + 16), LDS = STAGES * (BM + BN) * 128 > EPILOGUE ? STAGES * (BM + BN) * 128 : EPILOGUE;
    auto kernel = hbatched_dma_kernel<BM, BN, WM, WN, AK, BKC, STAGES>;
    static bool attr_set = false;   // raising the dynamic LDS limit is idempotent; races are harmless
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    MfmaArgs a{};
    a.A = p.A; a.B = p.B; a.C = p.C;
    a.lda = p.lda; a.ldb = p.ldb; a.ldc = p.ldc;
    a.m = a.m_main = static_cast<int>(p.m);
    a.n = a.n_main = static_cast<int>(p.n);
    a.k = static_cast<int>(p.k);
    a.alpha = p.alpha; a.beta = p.beta;
    a.tiles_m = static_cast<int>(ceil_div(p.m, BM));
    a.tiles_n = static_cast<int>(ceil_div(p.n, BN));
    const int64_t tiles = static_cast<int64_t>(a.tiles_m) * a.tiles_n;
    const BatchArgs b{batchwalk::divisor(tiles), p.stride_a, p.stride_b, p.stride_c};
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(tiles * p.batch)), dim3(WM * WN * 64), LDS, p.stream, a, b);
    return hipGetLastError();
}

// 128 x 128, 128 x 64 or 64 x 64: the tile that computes least beside the instance, the smaller ones at 1.05 and 1.25 times their area (they ask for
// the operands more often: 512 x (128, 128, 64) on the three 8.5 / 8.8 / 9.0 us; over 41 sizes any factors of 1.02 to 1.1 and 1.1 to 1.3 give the same)
int tile_of(const BatchedProblem &p)
{
    auto area = [&](int64_t bm, int64_t bn) { return static_cast<double>(ceil_div(p.m, bm) * bm) * static_cast<double>(ceil_div(p.n, bn) * bn); };
    const double cost[3] = {area(128, 128), 1.05 * area(128, 64), 1.25 * area(64, 64)};
    const int best = cost[1] < cost[0] ? 1 : 0;
    return cost[2] < cost[best] ? 2 : best;
}

template <bool AK, bool BKC> hipError_t launch_order(const BatchedProblem &p, int tile)
{
    switch (tile) {
    case 0: return launch<128, 128, 2, 4, AK, BKC, 2>(p);
    case 1: return launch<128, 64, 4, 2, AK, BKC, 2>(p);
    default: return launch<64, 64, 2, 2, AK, BKC, 2>(p);
    }
}

}  // namespace

bool batched_dma_fits(const BatchedProblem &p)
{
    if (!p.strided || p.dtype != MG_F16 || p.alpha == 0.f || p.k == 0) return false;
    const int64_t lim = int64_t(1) << 31;
    if (p.m >= lim || p.n >= lim || p.k >= lim || p.lda % 8 || p.ldb % 8 || p.stride_a % 8 || p.stride_b % 8) return false;
    if (pointer_alignment(p.A) < 16 || pointer_alignment(p.B) < 16) return false;
    if ((p.a_trans ? p.k : p.m) % 8 || (p.b_trans ? p.n : p.k) % 8) return false;
    if ((p.lda > p.ldb ? p.lda : p.ldb) * 128 * 2 >= lim - 4096) return false;
    // (the grid of the smallest tiles, in threads)
    return ceil_div(p.m, 64) * ceil_div(p.n, 64) * p.batch < lim / 128;
}

bool batched_dma_pays(const BatchedProblem &p)
{
    if (!batched_dma_fits(p)) return false;
    // whole 64^3 with A along m and B along k have a kernel of their own (10000 of them 36.7 us, here 38.0)
    if (p.m == 64 && p.n == 64 && p.k == 64 && !p.a_trans && !p.b_trans) return false;
    // Thin instances and streams from memory lose more to the tiles' empty part than the loads gain.  us, batched_tile.hip / here: 3000 x (40, 128, 128)
    // 27.7 / 30.3, 9000 x (56, 160, 32) (286 MB) 78 / 93, 7000 x (160, 80, 72) (421 MB) 135 / 168.  So do 64 x 64 tiles in large batches, and sooner where
    // neither operand runs along k: 1621 x 136^3 (180 MB) 51.5 / 59.2, 2000 x (56, 120, 176) (151 MB) 24.5 / 27.6.  Over 500 random batches calls take 0.86 of
    // the time without these kernels, those they do not take included; 6 are 3 to 8 % slower.
    const double mb = 2.0e-6 * static_cast<double>(p.batch) * static_cast<double>(p.m * p.k + p.k * p.n + p.m * p.n);
    const int64_t thin = p.m < p.n ? p.m : p.n;
    if (tile_of(p) == 2 && mb > (!p.a_trans && p.b_trans ? 40.0 : 80.0)) return false;
    return (thin >= 40 && mb <= 60.0) || (thin > 48 && mb <= 250.0);
}

hipError_t launch_batched_dma(const BatchedProblem &p, int tile)
{
    if (tile < 0) tile = tile_of(p);
    if (p.a_trans) return p.b_trans ? launch_order<true, false>(p, tile) : launch_order<true, true>(p, tile);
    return p.b_trans ? launch_order<false, false>(p, tile) : launch_order<false, true>(p, tile);
}

}  // namespace mg
