"""The kernel whose eight wavefronts share the sum of one 32 x 32 block (csrc/tiny.hip): sums beside its pairs of K-steps and beside eight of them, blocks
that end anywhere, pieces that would run past an operand's last line, all operand orders and alignments, against the CPU oracle, bit for bit on
integers."""
import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, N, T = W.COL_MAJOR, W.NO_TRANS, W.TRANS
ORDERS = {"mk": (N, N), "kk": (T, N), "mn": (N, T), "kn": (T, T)}


@pytest.mark.parametrize("order", sorted(ORDERS))
@pytest.mark.parametrize("dtype,pair", [("f32", 32), ("f16", 64)])
@pytest.mark.parametrize("m,n,pairs,over,pad", [(32, 32, 1, 0, 0), (35, 29, 1, 0, 0), (3, 5, 0, 1, 0), (33, 64, 1, -1, 1), (64, 31, 8, 1, 3), (40, 48, 9, 0, 8),
                                                (7, 100, 7, 5, 1), (65, 33, 41, -7, 0), (16, 70, 16, 0, 2)])
def test_blocks_and_pairs(oracle, dtype, pair, order, m, n, pairs, over, pad):
    """(what lies between and behind the lines of A and B is NaN)"""
    ta, tb = ORDERS[order]
    k = pairs * pair + over
    lds = dict(lda=W.tight_ld(C, ta, m, k) + pad, ldb=W.tight_ld(C, tb, k, n) + pad, ldc=m + pad)
    if dtype == "f32":
        import numpy as np
        g = W.rng_for(5, 31)
        matrices = (W.small_ints(g, s, 2, np.float32) for s in ((m, k), (k, n), (m, n)))
        case = W.make_case(f"shared_{m}x{n}x{k}", "f32", C, ta, tb, *matrices, 1.0, 1.0, exact=True, **lds)
    else:
        case = W.hgemm_case(m, n, k, case=31, layout=C, ta=ta, tb=tb, beta=1.0, integer=True, **lds)
    try:
        G.mg_override_config(G.kernel_id(("s" if dtype == "f32" else "h") + "tiny_32x32_" + order), 1)
        H.check_case(case, oracle)
    finally:
        G.mg_clear_override()


@pytest.mark.parametrize("order", sorted(ORDERS))
@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_beta_zero_leaves_nan_behind(oracle, dtype, order):
    import numpy as np
    ta, tb = ORDERS[order]
    case = (W.skinny_case(45, 50, 201, case=3, integer=True, ta=ta, tb=tb, alpha=2.0, beta=0.0) if dtype == "f32"
            else W.hgemm_case(45, 50, 201, case=3, ta=ta, tb=tb, beta=0.0, integer=True))
    case.C[:] = np.nan
    try:
        G.mg_override_config(G.kernel_id(("s" if dtype == "f32" else "h") + "tiny_32x32_" + order), 1)
        H.check_case(case, oracle)
    finally:
        G.mg_clear_override()


@pytest.mark.parametrize("order", sorted(ORDERS))
@pytest.mark.parametrize("k", [64, 96, 160, 288])
def test_error_of_a_sum_shared_by_eight(order, k):
    """FP32 error against 64 bits: at most that of eight equal parts of the sum, each added up term by term, and then each other's sums.

    The parts are added up here with one rounding per term; the tenth on top is for another order of the terms.  Chains of 32 terms, on
    as few wavefronts as that takes, have 1.36 times this error at k = 64 and 1.21 times at 288."""
    import numpy as np
    import torch
    ta, tb = ORDERS[order]
    rng = np.random.default_rng(7)
    a = (rng.random((256, k)) * 2 - 1).astype(np.float32)
    b = (rng.random((k, 256)) * 2 - 1).astype(np.float32)
    exact = a.astype(np.float64) @ b.astype(np.float64)
    total = np.zeros((256, 256), np.float32)
    for part in np.array_split(np.arange(k), 8):
        s = np.zeros((256, 256), np.float32)
        for l in part:
            s = (s.astype(np.float64) + np.outer(a[:, l].astype(np.float64), b[l].astype(np.float64))).astype(np.float32)
        total += s
    stored_a = torch.from_numpy(np.ascontiguousarray(a if ta == T else a.T)).cuda()
    stored_b = torch.from_numpy(np.ascontiguousarray(b if tb == T else b.T)).cuda()
    c = torch.zeros(256, 256, device="cuda")
    try:
        G.mg_override_config(G.kernel_id("stiny_32x32_" + order), 1)
        G.mg_sgemm(C, ta, tb, 256, 256, k, 1.0, stored_a, k if ta == T else 256, stored_b, 256 if tb == T else k, 0.0, c, 256, None)
    finally:
        G.mg_clear_override()
    error = lambda x: np.linalg.norm(x.astype(np.float64) - exact) / np.linalg.norm(exact)
    assert error(c.cpu().numpy().T) <= 1.1 * error(total)


@pytest.mark.parametrize("order", ["mk", "mn", "kn"])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("m,n", [(1, 33), (2, 40), (3, 5), (4, 2), (40, 3), (33, 1)])
@pytest.mark.parametrize("k,pad", [(64, 0), (65, 0), (66, 0), (70, 1), (129, 0), (577, 0), (130, 2)])
def test_lines_shorter_than_a_piece(oracle, dtype, order, m, n, k, pad):
    """operands along their rows of one to four rows, with next to nothing between the lines: the values that are left fill a pair and more"""
    import numpy as np
    ta, tb = ORDERS[order]
    rng = np.random.default_rng(m * 131 + n * 17 + k)
    draw = lambda *shape: rng.integers(-2, 3, shape)                # noqa: E731
    case = W.make_case(f"short_lines_{m}x{n}x{k}", dtype, C, ta, tb, draw(m, k), draw(k, n), draw(m, n), 1.0, 1.0,
                       W.tight_ld(C, ta, m, k) + pad, W.tight_ld(C, tb, k, n) + pad, m + pad, exact=True)
    try:
        G.mg_override_config(G.kernel_id(("s" if dtype == "f32" else "h") + "tiny_32x32_" + order), 1)
        H.check_case(case, oracle)
    finally:
        G.mg_clear_override()
