"""FP32 products with a short sum on the flavour that asks for C early (csrc/mfma_kernel.h): one to seven K-tiles, whole and partial,
edges of the tiles, every operand order, against the CPU oracle, bit for bit on integers."""
import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, R, N, T = W.COL_MAJOR, W.ROW_MAJOR, W.NO_TRANS, W.TRANS


@pytest.mark.parametrize("layout,ta,tb", [(C, N, N), (C, T, N), (C, N, T), (C, T, T), (R, N, T)])
@pytest.mark.parametrize("m,n", [(128, 64), (256, 192), (129, 65), (67, 131)])
@pytest.mark.parametrize("k", [1, 31, 32, 33, 64, 96, 100, 128, 192, 224])
def test_every_ending_of_the_sum_is_exact(oracle, layout, ta, tb, m, n, k):
    cm, cn = (m, n) if layout == C else (n, m)                           # as the column-major kernels see it
    whole = [tm for tm in (128, 64) if cm % tm == 0 and cn % 64 == 0 and k % 32 == 0]
    for beta in (0.0, -1.0):
        ran = 0
        case = W.skinny_case(m, n, k, case=m + k, integer=True, layout=layout, ta=ta, tb=tb, alpha=2.0, beta=beta)
        try:
            for t in G.kernel_table():
                if t["name"].startswith(("smfma_128x64x32_w2x2", "smfma_64x64x32_w2x2")):
                    G.mg_override_config(t["kernel_id"], 1)
                    try:
                        H.check_case(case, oracle)
                        ran += 1
                    except G.MgError as e:
                        assert e.status == -11                       # another operand order, or whole tiles only
        finally:
            G.mg_clear_override()
        assert ran == 2 + len(whole)                                     # the bounds-checked flavours, and those for whole tiles
        H.check_case(case, oracle)
