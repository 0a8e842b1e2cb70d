// Direct-to-LDS FP16 kernels for sizes that end inside a tile, on 16x16 MFMA blocks: operands whose rows start on 16 bytes and whose pieces
// of eight elements lie wholly inside or outside (dma_ragged_operands in internal.h).  Such problems ran on the register-staged kernels, in
// place or in slices, whose loads are two K-tiles ahead at most and whose larger tiles leave much of the last turn of tiles idle.
//   * 192 x 192 (three stages, 144 KB), bound by the matrix pipes at the power limit: between 128 x 128 and 256 x 256, whole tiles too: a
//     square of 3072 is 256 tiles of it, one turn (256 x 256: 144; us, best of the other kernels / this one: 3072^3 57.8 / 50.7, 3000^3
//     68.5 / 51.4), SYRK 4096 253 of a triangle's tiles (256 x 256: 136 tiles, 83.4 / 69.4).  Eight wavefronts of 96 x 48; four of 96 x 96, one
//     per SIMD, read a third less of LDS but cover no waits: 3072^3 57.8, 4096^3 141 against 122.
//   * 192 x 128 and 128 x 128 (four stages, 160 and 128 KB): 2056^3 37.7 / 26.3, 1536^3 (whole tiles) 13.1 / 13.2.
//   * 128 x 64 and 64 x 64 (four stages, 96 and 64 KB): bound by the latency of their loads, 0.16 us per K-tile; one turn of them takes
//     what the register-staged tiles need slices and a second launch for: (1672, 560, 3264) 20.3 / 15.3, (448, 608, 2744) 13.8 / 11.3.
// 256 x 256 in this flavour spills up to 67 registers and 256 x 128 is the fastest on 13 of 190 sizes by 0.1 % in the mean: left out.
// Over 190 sizes of 64 to 6000 in all orders the best of these tiles is 1.19 times (geometric mean) as fast as the kernels they replace.
#include "mfma_dma_host.h"
namespace mg {
#define MG_RAGGED(tag, BM, BN, WM, WN, STAGES)                                                 \
    table.push_back(MfmaRaggedConfig<BM, BN, WM, WN, true, true, STAGES>::entry(tag "_kk"));   \
    table.push_back(MfmaRaggedConfig<BM, BN, WM, WN, false, true, STAGES>::entry(tag "_mk"));  \
    table.push_back(MfmaRaggedConfig<BM, BN, WM, WN, true, false, STAGES>::entry(tag "_kn"));  \
    table.push_back(MfmaRaggedConfig<BM, BN, WM, WN, false, false, STAGES>::entry(tag "_mn"));
void register_hdma16r(std::vector<KernelEntry> &table)
{
    MG_RAGGED("hdma16r_192x192x64_w2x4", 192, 192, 2, 4, 3)
    MG_RAGGED("hdma16r_192x128x64_w2x4", 192, 128, 2, 4, 4)
    MG_RAGGED("hdma16r_128x128x64_w2x4", 128, 128, 2, 4, 4)
    MG_RAGGED("hdma16r_128x64x64_w4x2", 128, 64, 4, 2, 4)
    MG_RAGGED("hdma16r_64x64x64_w2x2", 64, 64, 2, 2, 4)
}
}  // namespace mg
