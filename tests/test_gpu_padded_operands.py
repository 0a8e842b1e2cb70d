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


def _kernels(case):
    """names of the kernels that one call of the case launches"""
    import torch
    from torch.profiler import ProfilerActivity, profile
    from paper_1705_05249_amd import gemm as G
    A, B, Cm = H.to_gpu(case.A), H.to_gpu(case.B), H.to_gpu(case.C)
    ws = H.workspace_for(case)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as record:
        G.mg_hgemm(case.layout, case.ta, case.tb, case.m, case.n, case.k, case.alpha, A, case.lda, B, case.ldb, case.beta, Cm, case.ldc, ws)
        torch.cuda.synchronize()
    return [e.name for e in record.events() if "mg::" in e.name or "_ZN2mg" in e.name]


@pytest.mark.parametrize("ta,tb", [(N, N), (T, N), (N, T), (T, T)])
@pytest.mark.parametrize("m,n,tile,ktiles", [(1995, 1611, "128, 128, 2, 4", t) for t in (17, 18, 19, 20)] +
                         [(2177, 2051, "256, 128, 4, 2", t) for t in (12, 13, 14)])
def test_every_remainder_of_the_staged_loops(oracle, ta, tb, m, n, tile, ktiles):
    """every number of K-tiles modulo three and modulo four, on the kernel with three (256 x 128) or four (128 x 128) stages"""
    odd = lambda x: x + (x % 2 == 0)                                 # noqa: E731
    k = 64 * ktiles - 7
    case = W.hgemm_case(m, n, k, case=m + k, layout=C, ta=ta, tb=tb, alpha=1.0, beta=1.0, integer=True,
                        lda=odd(W.tight_ld(C, ta, m, k)), ldb=odd(W.tight_ld(C, tb, k, n)), ldc=odd(m))
    H.check_case(case, oracle)
    ran = _kernels(case)
    stages = 4 if tile.startswith("128") else 3
    order = f"{'true' if ta == T else 'false'}, {'true' if tb == N else 'false'}"
    assert any(f"hgemm_dma_kernel<{tile}, {order}, 16, 0, true, {stages}>" in name for name in ran), ran


@pytest.mark.parametrize("ta,tb", [(N, N), (T, N), (N, T), (T, T)])
def test_short_sums_of_small_products_stay_in_place(oracle, ta, tb):
    """rows at odd elements, 1301 terms: 19 us in place, 22 through the copies"""
    case = W.hgemm_case(1301, 1301, 1301, case=3, layout=C, ta=ta, tb=tb, alpha=1.0, beta=1.0, integer=True)
    H.check_case(case, oracle)
    assert not any("pad_matrices" in name for name in _kernels(case))
