"""The direct-to-LDS FP16 kernels for sizes that end inside a tile (csrc/mfma_dma_kernel.h, DMA_RAGGED): one 16-byte piece short of a tile, one
over it, single pieces, sums shorter than the pipeline, all operand orders, slices, triangles of C, against the CPU oracle, bit for bit on
integers; what lies between the columns is NaN in A and B and stays as it was in C."""
import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, N, T = W.COL_MAJOR, W.NO_TRANS, W.TRANS
TILES = [(192, 192), (192, 128), (128, 128), (128, 64), (64, 64)]
ORDERS = {"mk": (N, N), "kk": (T, N), "mn": (N, T), "kn": (T, T)}


def kernel(tile, order):
    name, = [t["name"] for t in G.kernel_table() if t["name"].startswith(f"hdma16r_{tile[0]}x{tile[1]}x64_") and t["name"].endswith("_" + order)]
    return G.kernel_id(name)


def up8(x):
    return -(-x // 8) * 8 + 8


@pytest.mark.parametrize("order", sorted(ORDERS))
@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("dm,dn,k,slices", [(0, 0, 64, 1), (-8, 8, 8, 1), (8, -8, 72, 1), (8, 8, 184, 2), (-8, -8, 248, 1), (16, 0, 328, 3), (None, None, 392, 1)])
def test_sizes_beside_a_tile(oracle, tile, order, dm, dn, k, slices):
    """dm, dn: beside one tile (None: a single 16-byte piece)"""
    ta, tb = ORDERS[order]
    m, n = (tile[0] + dm, tile[1] + dn) if dm is not None else (8, 8)
    # the direction that no piece runs along may have any length
    if order[0] == "k":
        m -= 3
    if order[1] == "k":
        n -= 5
    case = W.hgemm_case(m, n, k, case=m + k, layout=C, ta=ta, tb=tb, alpha=1.0, beta=float(slices % 2), integer=True,
                        lda=up8(W.tight_ld(C, ta, m, k)), ldb=up8(W.tight_ld(C, tb, k, n)), ldc=m + 3)
    import torch
    workspace = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")
    try:
        G.mg_override_config(kernel(tile, order), slices)
        H.check_case(case, oracle, workspace=workspace)
    finally:
        G.mg_clear_override()


def test_operands_whose_pieces_end_outside_are_refused():
    """rows off 16 bytes, a piece that ends inside an operand: no kernel of the family (and another one takes the call)"""
    for m, n, k, lda, ldb, order in ((192, 192, 68, 72, 72, "kk"), (100, 192, 64, 104, 64, "mk"), (192, 192, 64, 68, 64, "kk"), (192, 100, 64, 192, 104, "mn")):
        ta, tb = ORDERS[order]
        try:
            G.mg_override_config(kernel((192, 192), order), 1)
            assert G.lib().mg_query_selected(G.MG_F16, C, ta, tb, m, n, k, lda, ldb, m, 1.0, 0.0, 256, G.mg_config()) == -11
        finally:
            G.mg_clear_override()
        assert not G.mg_query_selected(G.MG_F16, C, ta, tb, m, n, k, lda, ldb, m)["name"].startswith("hdma16r")


@pytest.mark.parametrize("tile", [(192, 192), (128, 128), (64, 64)])
@pytest.mark.parametrize("uplo", [W.UPPER, W.LOWER])
@pytest.mark.parametrize("tiles,trans,slices", [(1, N, 1), (3, T, 1), (8, N, 2), (10, T, 1)])
def test_triangles_of_c(level3_oracle, tile, uplo, tiles, trans, slices):
    n = tiles * tile[0] - 8
    case = W.level3_case("syrk", "f16", C, n, n, k=136, uplo=uplo, trans=trans, alpha=1.0, beta=-1.0, integer=True, case=n)
    import torch
    workspace = torch.empty(256 + 2 * n * n + 4 * slices * n * n, dtype=torch.uint8, device="cuda")
    try:
        G.mg_override_config(kernel(tile, "mn" if trans == N else "kk"), slices)
        H.check_level3(case, level3_oracle, workspace=workspace)
    finally:
        G.mg_clear_override()
