"""The direct-to-LDS FP16 kernels with three and four LDS stages (csrc/mfma_dma_kernel.h): sums shorter than the pipeline and every
remainder of the unrolled loop, all operand orders, beta, sliced sums, against the CPU oracle, bit for bit on integers."""
import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, R, N, T = W.COL_MAJOR, W.ROW_MAJOR, W.NO_TRANS, W.TRANS


@pytest.mark.parametrize("ta,tb", [(N, N), (T, N), (N, T), (T, T)])
@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 6, 7, 8, 9])
def test_every_length_of_the_loop_is_exact(oracle, ta, tb, tiles):
    case = W.hgemm_case(256, 384, 64 * tiles, case=tiles, layout=C, ta=ta, tb=tb, alpha=1.0, beta=float(tiles % 2), integer=True)
    ran = 0
    try:
        for t in G.kernel_table():
            if t["name"].startswith(("hdeep16_", "hdma16_256x128")):
                for slices in (1, 2):
                    G.mg_override_config(t["kernel_id"], slices)
                    try:
                        H.check_case(case, oracle)
                        ran += 1
                    except G.MgError as e:
                        assert e.status == -11               # another operand order, or an empty slice
    finally:
        G.mg_clear_override()
    assert ran >= 2
