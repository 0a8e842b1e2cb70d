"""Products of 2 to 15 rows or columns, whose sums are longer than one block's wavefronts share or which have more blocks than the chip has compute
units: with the workspace the library asks for and without, against the CPU oracle."""
import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, R, N, T = W.COL_MAJOR, W.ROW_MAJOR, W.NO_TRANS, W.TRANS


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("layout,ta,tb", [(C, N, N), (C, T, N), (C, N, T), (R, T, T)])
@pytest.mark.parametrize("m,n,k", [(2, 2, 4001), (3, 9001, 70), (8, 8, 2600), (8, 8300, 49), (15, 37, 3000), (500, 7, 1700), (5, 8209, 129)])
@pytest.mark.parametrize("workspace", ["auto", None])
def test_thin(oracle, dtype, layout, ta, tb, m, n, k, workspace):
    case = (W.skinny_case if dtype == "f32" else W.hgemm_case)(m, n, k, case=m + n + k, layout=layout, ta=ta, tb=tb, beta=0.5)
    H.check_case(case, oracle, workspace=workspace)
    args = (G.MG_F32 if dtype == "f32" else G.MG_F16, layout, ta, tb, m, n, k, case.lda, case.ldb, case.ldc)
    assert not G.mg_kernel_name(G.mg_query_selected(*args)["kernel_id"]).startswith("direct")


@pytest.mark.parametrize("layout,ta,tb,m,n,k", [(C, N, N, 7, 9000, 700), (C, T, N, 7, 9000, 700), (R, T, T, 12001, 7, 1001), (C, N, T, 4, 30000, 400)])
def test_fewer_than_eight_rows_share_their_sums(oracle, layout, ta, tb, m, n, k):
    """no 256 x 256 tile for them: (7, 9000, 700) 54.7 / 12.2 us"""
    case = W.hgemm_case(m, n, k, case=m + n + k, layout=layout, ta=ta, tb=tb, beta=0.5)
    sel = G.mg_query_selected(G.MG_F16, layout, ta, tb, m, n, k, case.lda, case.ldb, case.ldc)
    assert G.mg_kernel_name(sel["kernel_id"]).startswith("htiny_32x32")
    H.check_case(case, oracle)


def test_static_scratch_takes_the_slices_that_fit():
    """17 MB of partial sums would be preferred, the array holds 16; integers, exact"""
    import torch
    m, n, k = 35500, 15, 4000
    assert G.mg_gemm_workspace_bytes(G.MG_F32, C, N, N, m, n, k, m, k, m) > G.MG_STATIC_SCRATCH_BYTES
    gen = torch.Generator(device="cuda").manual_seed(1)
    A = torch.randint(-2, 3, (k, m), device="cuda", generator=gen).float()
    B = torch.randint(-2, 3, (n, k), device="cuda", generator=gen).float()
    out = torch.full((n, m), float("nan"), device="cuda")
    G.mg_sgemm_static(C, N, N, m, n, k, 1.0, A, m, B, k, 0.0, out, m)
    assert torch.equal(out.double(), B.double() @ A.double())
