"""Triangles on the shared-sum kernel (csrc/tiny.hip): SYRK, which writes the wanted triangle only, and TRMM, whose sums end or begin with the
block's rows, at the edges of its 32 x 32 blocks and pairs of K-steps, against the CPU oracle, bit for bit on integers."""
import itertools

import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

R, C, N, T = W.ROW_MAJOR, W.COL_MAJOR, W.NO_TRANS, W.TRANS
UP, LO, LEFT, RIGHT = W.UPPER, W.LOWER, W.LEFT, W.RIGHT


def forced(case, level3_oracle, dtype):
    """automatic selection, then every order of the kernel"""
    H.check_level3(case, level3_oracle)
    ran = 0
    try:
        for t in G.kernel_table():
            if t["name"].startswith("stiny" if dtype == "f32" else "htiny"):
                G.mg_override_config(t["kernel_id"], 1)
                try:
                    H.check_level3(case, level3_oracle)
                    ran += 1
                except G.MgError as e:
                    assert e.status == -11               # another operand order
    finally:
        G.mg_clear_override()
    assert ran == 1


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("layout,uplo,trans", list(itertools.product([C, R], [UP, LO], [N, T])))
@pytest.mark.parametrize("n,k,pad", [(2, 48, 0), (31, 63, 1), (33, 64, 0), (64, 513, 3), (97, 200, 0), (705, 70, 1)])
def test_syrk(level3_oracle, dtype, layout, uplo, trans, n, k, pad):
    forced(W.level3_case("syrk", dtype, layout, n, n, k=k, uplo=uplo, trans=trans, alpha=2.0, beta=-1.0, pad=(pad, 0, 2 * pad), case=n + k,
                         integer=True), level3_oracle, dtype)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("layout,uplo,side,trans", list(itertools.product([C, R], [UP, LO], [LEFT, RIGHT], [N, T])))
@pytest.mark.parametrize("m,n,pad", [(33, 2, 0), (31, 65, 1), (64, 96, 0), (100, 161, 3)])
def test_trmm(level3_oracle, dtype, layout, uplo, side, trans, m, n, pad):
    forced(W.level3_case("trmm", dtype, layout, m, n, side=side, uplo=uplo, trans=trans, alpha=2.0, pad=(pad, 2 * pad, 0), case=m + n,
                         integer=True), level3_oracle, dtype)
