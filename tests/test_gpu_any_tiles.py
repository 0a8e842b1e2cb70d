"""The FP16 kernels whose pieces come from any element (csrc/mfma_any_kernel.h): sizes one short of a tile, one over it and below a piece's length
beyond one, leading dimensions and pointers at odd elements, sums shorter than the pipeline and sums that end inside a piece, all
operand orders, slices, triangles of C and of an operand, against the CPU oracle, bit for bit on integers; what lies between the columns is NaN in A and B and
stays as it was in C."""
import itertools

import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, N, T = W.COL_MAJOR, W.NO_TRANS, W.TRANS
TILES = [(256, 128), (192, 128), (128, 128), (128, 64), (64, 64)]
ORDERS = {"mk": (N, N), "kk": (T, N), "mn": (N, T), "kn": (T, T)}


def kernel(tile, order):
    name, = [t["name"] for t in G.kernel_table() if t["name"].startswith(f"hany16_{tile[0]}x{tile[1]}x64_") and t["name"].endswith("_" + order)]
    return G.kernel_id(name)


@pytest.mark.parametrize("order", sorted(ORDERS))
@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("dm,dn,k,slices,pad", [(0, 0, 8, 1, 0), (-1, 1, 63, 1, 0), (1, -1, 65, 1, 1), (7, 9, 129, 1, 0), (-9, -7, 193, 2, 1), (3, 5, 257, 1, 2),
                                                (0, 0, 320, 1, 1), (64, 1, 385, 4, 0), (None, None, 71, 1, 1)])
def test_sizes_beside_a_tile(oracle, tile, order, dm, dn, k, slices, pad):
    """dm, dn: beside one tile (None: eight rows and columns, the fewest); pad: elements between the columns of A and B"""
    ta, tb = ORDERS[order]
    m, n = (tile[0] + dm, tile[1] + dn) if dm is not None else (8, 8)
    case = W.hgemm_case(m, n, k, case=m + k, layout=C, ta=ta, tb=tb, alpha=1.0, beta=float(k % 2), integer=True,
                        lda=W.tight_ld(C, ta, m, k) + pad, ldb=W.tight_ld(C, tb, k, n) + pad, ldc=m + pad)
    import torch
    workspace = torch.empty(4 * slices * m * n + 256, dtype=torch.uint8, device="cuda")
    try:
        G.mg_override_config(kernel(tile, order), slices)
        H.check_case(case, oracle, workspace=workspace)
    finally:
        G.mg_clear_override()


@pytest.mark.parametrize("order", sorted(ORDERS))
@pytest.mark.parametrize("m,n,k", [(129, 70, 100), (65, 64, 64), (200, 9, 200)])
def test_matrices_that_end_with_their_buffers(order, m, n, k):
    """Operands at odd elements whose last element is the last before a NaN: what is read beside a matrix never counts, and nothing is
    written there.  FP16 results of sums of k products against FP64: 2^-11 of the value and k roundings to FP32 of the absolute sum."""
    import torch
    ta, tb = ORDERS[order]
    gen = torch.Generator(device="cuda").manual_seed(m + k)

    def matrix(rows, cols, at):
        buffer = torch.full((at + rows * cols + 16,), float("nan"), dtype=torch.float16, device="cuda")
        inside = buffer[at:at + rows * cols].view(cols, rows)
        inside.copy_(torch.randn(cols, rows, device="cuda", generator=gen))
        return buffer, inside.T
    A, a = matrix(*W.stored_extents(ta, m, k), 3)
    B, b = matrix(*W.stored_extents(tb, k, n), 5)
    a, b = (x.double() if t == N else x.T.double() for x, t in ((a, ta), (b, tb)))
    want, size = a @ b, a.abs() @ b.abs()
    for tile in TILES:
        out, c = matrix(m, n, 7)
        try:
            G.mg_override_config(kernel(tile, order), 1)
            G.mg_hgemm(C, ta, tb, m, n, k, 1.0, A.data_ptr() + 6, W.tight_ld(C, ta, m, k), B.data_ptr() + 10, W.tight_ld(C, tb, k, n), 0.0,
                       out.data_ptr() + 14, m)
        finally:
            G.mg_clear_override()
        assert bool(((c.double() - want).abs() <= 2.0 ** -11 * want.abs() + 2.0 ** -24 * k * size + 2.0 ** -25).all()), tile
        assert bool(out[:7].isnan().all()) and bool(out[7 + m * n:].isnan().all())


@pytest.mark.parametrize("tile", [(128, 128), (64, 64)])
@pytest.mark.parametrize("uplo", [W.UPPER, W.LOWER])
@pytest.mark.parametrize("tiles,trans,slices,beta", [(1, N, 1, -1.0), (3, T, 1, 0.0), (5, N, 2, -1.0), (6, T, 1, -1.0)])
def test_triangles_of_c(level3_oracle, tile, uplo, tiles, trans, slices, beta):
    n = tiles * tile[0] - 3
    case = W.level3_case("syrk", "f16", C, n, n, k=137, uplo=uplo, trans=trans, alpha=1.0, beta=beta, integer=True, case=n)
    import torch
    workspace = torch.empty(256 + 2 * n * n + 4 * slices * n * n, dtype=torch.uint8, device="cuda")
    try:
        G.mg_override_config(kernel(tile, "mn" if trans == N else "kk"), slices)
        H.check_level3(case, level3_oracle, workspace=workspace)
    finally:
        G.mg_clear_override()


@pytest.mark.parametrize("layout,side,uplo,trans", list(itertools.product([C, W.ROW_MAJOR], [W.LEFT, W.RIGHT], [W.UPPER, W.LOWER], [N, T])))
@pytest.mark.parametrize("m,n", [(641, 9), (70, 401), (129, 193), (401, 209)])
def test_triangular_operands(level3_oracle, layout, side, uplo, trans, m, n):
    """TRMM on every tile, one to four slices, of which those wholly among the operand's zeros add nothing"""
    import torch
    case = W.level3_case("trmm", "f16", layout, m, n, side=side, uplo=uplo, trans=trans, alpha=1.0, integer=True, case=m + n)
    workspace = torch.empty((m + n) * (m + n + 64) * 4 + 4 * 4 * m * n + 4096, dtype=torch.uint8, device="cuda")
    ran = set()
    try:
        for t in G.kernel_table():
            if not t["name"].startswith("hany16"):
                continue
            for slices in (1, 2, 4):
                G.mg_override_config(t["kernel_id"], slices)
                try:
                    H.check_level3(case, level3_oracle, workspace=workspace)
                    ran.add((t["name"].rsplit("_", 1)[0], slices))
                except G.MgError as e:
                    assert e.status == -11               # another operand order, an empty slice
    finally:
        G.mg_clear_override()
    longest = m if side == W.LEFT else n
    assert len({name for name, slices in ran if slices == 1}) == 5 and (longest < 193 or len({name for name, slices in ran if slices == 4}) == 5), ran


@pytest.mark.parametrize("layout,side,uplo,trans", [(C, W.LEFT, W.LOWER, N), (C, W.RIGHT, W.UPPER, T), (W.ROW_MAJOR, W.LEFT, W.UPPER, T), (W.ROW_MAJOR, W.RIGHT, W.LOWER, N)])
def test_triangular_operands_of_odd_sizes(level3_oracle, layout, side, uplo, trans):
    """more blocks than the shared-sum kernel takes, sums beyond the register-staged tiles: what selection chooses"""
    m, n = (1001, 303) if side == W.LEFT else (303, 1001)
    H.check_level3(W.level3_case("trmm", "f16", layout, m, n, side=side, uplo=uplo, trans=trans, alpha=1.0, integer=True, case=m + n), level3_oracle)


@pytest.mark.parametrize("tile", [(128, 128), (64, 64)])
@pytest.mark.parametrize("uplo", [W.UPPER, W.LOWER])
@pytest.mark.parametrize("n", [61, 125, 131, 259])
def test_the_other_triangle_of_c_may_hold_anything(tile, uplo, n):
    """beta with NaN and infinities outside the wanted triangle, which stay as they are; integers, exact"""
    import torch
    k, ldc = 137, n + 3
    gen = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randint(-2, 3, (n, k), device="cuda", generator=gen).half()                     # row by row: n x k, contiguous along k
    want = torch.ones(n, n, dtype=torch.bool, device="cuda")
    want = want.tril() if uplo == W.LOWER else want.triu()
    before = torch.randint(-3, 4, (n, n), device="cuda", generator=gen).half()
    before[~want] = torch.tensor([float("nan"), float("inf")], device="cuda").half().repeat(n * n)[:int((~want).sum())]
    buffer = torch.full((n * ldc,), float("nan"), device="cuda", dtype=torch.float16)
    inside = buffer.view(n, ldc)[:, :n].T                                                      # column-major: inside[i, j]
    inside.copy_(before)
    workspace = torch.empty(G.mg_syrk_workspace_bytes(G.MG_F16, C, T, n, k) + 4 * n * n + 256, dtype=torch.uint8, device="cuda")
    try:
        G.mg_override_config(kernel(tile, "kk"), 1)
        G.mg_hsyrk(C, uplo, T, n, k, 1.0, A, k, -1.0, buffer, ldc, workspace)
    finally:
        G.mg_clear_override()
    after = torch.where(want, (A.double() @ A.double().T - before.double()).half(), before)
    bits = lambda x: x.contiguous().view(torch.int16)  # noqa: E731
    assert torch.equal(bits(inside), bits(after))
    assert bool(buffer.view(n, ldc)[:, n:].isnan().all())


def test_too_few_elements_for_a_piece_are_refused():
    for m, n, k in ((7, 64, 64), (64, 7, 64), (64, 64, 7)):
        try:
            G.mg_override_config(kernel((64, 64), "mk"), 1)
            assert G.lib().mg_query_selected(G.MG_F16, C, N, N, m, n, k, m, k, m, 1.0, 0.0, 2, G.mg_config()) == -11
        finally:
            G.mg_clear_override()


def test_off_16_bytes_they_take_longer_sums():
    """and the register-staged tiles sums of one K-tile into a large C"""
    assert G.mg_query_selected(G.MG_F16, C, N, N, 1501, 1501, 1501, 1505, 1505, 1505)["name"].startswith("hany16")
    assert G.mg_query_selected(G.MG_F16, C, N, N, 5306, 4288, 60, 5306, 60, 5306)["name"].startswith("hmfma")
