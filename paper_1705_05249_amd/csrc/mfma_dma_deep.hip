// Direct-to-LDS FP16 kernel on 128 x 128 tiles with four LDS stages, three K-tiles of loads in flight, for grids that give a
// compute unit one work-group at most.  With two stages a K-tile cannot take less than a load's latency (0.9 us where the matrix
// pipes need 0.21); with four it takes 0.3-0.45 us, and the one work-group uses 128 of the 160 KB of LDS that two of
// the two-stage kernel share.  us, best of the other kernels / this one: 2048^3 24.9 / 21.2 (A along m, B along n 27.8 / 22.7), 1536^3
// 18.1 / 14.7, 1024 x 2048 x 4096 30.2 / 26.8; 512 tiles: 4096 x 2048 x 1024 22.0 / 24.4.  (Four wavefronts of 64 x 64
// with three stages: 23.8, 17.7, 34.2.)
#include "mfma_dma_host.h"
namespace mg {
void register_hdeep16(std::vector<KernelEntry> &table)
{
    table.push_back(MfmaDmaConfig<128, 128, 2, 4, true, true, 16, false, 4>::entry("hdeep16_128x128x64_w2x4_kk"));
    table.push_back(MfmaDmaConfig<128, 128, 2, 4, false, true, 16, false, 4>::entry("hdeep16_128x128x64_w2x4_mk"));
    table.push_back(MfmaDmaConfig<128, 128, 2, 4, true, false, 16, false, 4>::entry("hdeep16_128x128x64_w2x4_kn"));
    table.push_back(MfmaDmaConfig<128, 128, 2, 4, false, false, 16, false, 4>::entry("hdeep16_128x128x64_w2x4_mn"));
}
}  // namespace mg
