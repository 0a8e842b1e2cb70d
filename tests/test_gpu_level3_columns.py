"""Dense operands of SYMM and TRMM in the workspace: columns that start on 16 bytes, and tight ones where the workspace has no room
for more, with sizes around the runs of 16 bytes, against the CPU oracle."""
import pytest

import helpers as H
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

R, C, N, T = W.ROW_MAJOR, W.COL_MAJOR, W.NO_TRANS, W.TRANS


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("routine", ["symm", "trmm"])
@pytest.mark.parametrize("layout,side,uplo", [(C, W.LEFT, W.LOWER), (R, W.RIGHT, W.UPPER), (C, W.RIGHT, W.UPPER), (R, W.LEFT, W.LOWER)])
@pytest.mark.parametrize("m,n", [(7, 9), (8, 15), (129, 127), (133, 260), (257, 31)])
def test_aligned_and_tight_columns(level3_oracle, dtype, routine, layout, side, uplo, m, n):
    import torch
    case = W.level3_case(routine, dtype, layout, m, n, side=side, uplo=uplo, alpha=2.0, beta=-1.0, pad=(1, 1, 1), integer=True, case=m + n)
    H.check_level3(case, level3_oracle)
    ka, size = (m if side == W.LEFT else n), 4 if dtype == "f32" else 2
    tight = (ka * ka * size + 255) // 256 * 256 + ((m * n * size + 255) // 256 * 256 if routine == "trmm" else 0)
    H.check_level3(case, level3_oracle, workspace=torch.empty(tight, dtype=torch.uint8, device="cuda"))
