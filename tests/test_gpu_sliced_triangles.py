"""Long sums over few outputs in the triangular routines: SYRK, whose slices are added up for the wanted triangle only, and TRMM, whose
slices hold tiles with nothing to add, against the CPU oracle, bit for bit on integers."""
import itertools

import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

R, C, N, T = W.ROW_MAJOR, W.COL_MAJOR, W.NO_TRANS, W.TRANS
UP, LO, LEFT, RIGHT = W.UPPER, W.LOWER, W.LEFT, W.RIGHT


def every_slicing(case, level3_oracle, prefixes):
    """automatic selection, then every kernel of these names with two and five slices; bytes outside the triangle stay"""
    import torch
    H.check_level3(case, level3_oracle)
    workspace = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    ran = 0
    try:
        for t in G.kernel_table():
            if t["name"].startswith(prefixes):
                for slices in (2, 5):
                    G.mg_override_config(t["kernel_id"], slices)
                    try:
                        H.check_level3(case, level3_oracle, workspace=workspace)
                        ran += 1
                    except G.MgError as e:
                        assert e.status == -11               # another operand order, whole tiles only, an empty slice
    finally:
        G.mg_clear_override()
    return ran


@pytest.mark.parametrize("dtype,prefixes", [("f32", ("smfma_64x64", "smfma_128x128", "ssplit")), ("f16", ("hmfma_64x64", "hmfma_256x128", "hdma16_128", "hdeep16", "hpp16_"))])
@pytest.mark.parametrize("layout,uplo", list(itertools.product([C, R], [UP, LO])))
@pytest.mark.parametrize("n,k", [(64, 1000), (129, 1030), (256, 1024), (258, 644)])
def test_sliced_syrk(level3_oracle, dtype, prefixes, layout, uplo, n, k):
    case = W.level3_case("syrk", dtype, layout, n, n, k=k, uplo=uplo, trans=T if n % 2 else N, alpha=1.0, beta=-1.0, pad=(0, 0, 2 * (n % 2)),
                         integer=True, case=n + k)
    assert every_slicing(case, level3_oracle, prefixes) >= 2


@pytest.mark.parametrize("dtype,prefixes", [("f32", ("smfma_64x64", "smfma_128x128", "ssplit")), ("f16", ("hmfma_64x64", "hmfma_256x128", "hdma16_128", "hdeep16", "hpp16_"))])
@pytest.mark.parametrize("layout,side,uplo,trans", [(C, LEFT, LO, N), (C, RIGHT, UP, T), (R, LEFT, UP, T), (R, RIGHT, LO, N)])
@pytest.mark.parametrize("m,n", [(640, 70), (70, 641), (768, 256), (256, 512)])
def test_sliced_trmm(level3_oracle, dtype, prefixes, layout, side, uplo, trans, m, n):
    case = W.level3_case("trmm", dtype, layout, m, n, side=side, uplo=uplo, trans=trans, alpha=1.0, integer=True, case=m + n)
    assert every_slicing(case, level3_oracle, prefixes) >= 2
