"""Ragged FP16 problems on padded copies of A and B with C in place (run_indirect in csrc/api.hip): the 256 x 128 and 128 x 128 tiles with
three and four LDS stages whose epilogue ends inside a tile, every operand order, odd and even leading dimensions, against the CPU
oracle; what lies beside C stays as it was."""
import pytest

import helpers as H
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, R, N, T = W.COL_MAJOR, W.ROW_MAJOR, W.NO_TRANS, W.TRANS


@pytest.mark.parametrize("ta,tb", [(N, N), (T, N), (N, T), (T, T)])
@pytest.mark.parametrize("m,n,k,layout,odd", [(1345, 1409, 1057, C, 1), (2177, 2051, 450, C, 1), (1283, 1290, 1280, R, 1), (1538, 1500, 1474, C, 2)])
def test_c_in_place(oracle, ta, tb, m, n, k, layout, odd):
    ld = lambda x: x + (x % 2 == 0 if odd == 1 else 2 - x % 2)       # noqa: E731  (odd, or even and not a multiple of the tile)
    case = W.hgemm_case(m, n, k, case=m + k, layout=layout, ta=ta, tb=tb, alpha=1.0, beta=1.0, integer=True,
                        lda=ld(W.tight_ld(layout, ta, m, k)), ldb=ld(W.tight_ld(layout, tb, k, n)), ldc=ld(W.tight_ld(layout, N, m, n)))
    H.check_case(case, oracle)
