"""FP32 kernels on the bf16 matrix pipes (csrc/mfma_split_kernel.h): edges of the tiles and of the sum, values that three bf16
parts cannot hold, and their error beside that of the kernels on the FP32 pipes."""
import numpy as np
import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, R, N, T = W.COL_MAJOR, W.ROW_MAJOR, W.NO_TRANS, W.TRANS


def forced(prefix, call, slices=1):
    """runs call() once for every kernel of that name that takes the problem"""
    ran = 0
    try:
        for t in G.kernel_table():
            if t["name"].startswith(prefix):
                G.mg_override_config(t["kernel_id"], slices)
                try:
                    call()
                    ran += 1
                except G.MgError as e:
                    assert e.status == -11                   # another operand order, whole tiles only, an empty slice
    finally:
        G.mg_clear_override()
    return ran


def wide_integers(g, shape):
    """19 bits, odd: most of them have all three parts"""
    return ((2 * g.integers(2 ** 17, 2 ** 18, shape) + 1) * g.choice([-1, 1], shape)).astype(np.float32)


def few_ones(g, rows, k):
    """rows x k, 1 and -1 at up to 31 places of each row"""
    out = np.zeros((rows, k), np.float32)
    for r in range(rows):
        at = g.choice(k, min(k, 31), replace=False)
        out[r, at] = g.choice([-1, 1], at.size)
    return out


# (row-major T, T: both operands along their rows after the swap, the one order that the others leave out)
@pytest.mark.parametrize("layout,ta,tb", [(C, N, N), (C, T, N), (C, N, T), (R, T, T)])
@pytest.mark.parametrize("m,n", [(256, 128), (257, 131), (63, 66), (5, 129), (130, 1)])
@pytest.mark.parametrize("k", [1, 15, 16, 17, 31, 32, 33, 64, 95, 96, 127, 128, 129, 160, 257, 400])
def test_every_edge_is_exact(oracle, layout, ta, tb, m, n, k):
    import torch
    workspace = torch.empty(2 * 4 * m * n, dtype=torch.uint8, device="cuda")
    case = W.skinny_case(m, n, k, case=m + k, integer=True, layout=layout, ta=ta, tb=tb, alpha=2.0, beta=float(k % 2))
    g = np.random.default_rng(m + n + k)
    cases = [case]
    # each part of one operand at its place: sums of up to 31 integers below 2^19, exact
    for a, b in ((wide_integers(g, (m, k)), few_ones(g, n, k).T), (few_ones(g, m, k), wide_integers(g, (k, n)))):
        cases.append(W.make_case(f"parts_{m}x{n}x{k}", "f32", layout, ta, tb, a, b, np.zeros((m, n), np.float32), 2.0, 0.0,
                                 case.lda, case.ldb, case.ldc, exact=True))
    for c in cases:
        assert forced("ssplit", lambda: H.check_case(c, oracle)) >= 2
        if k >= 64:
            assert forced("ssplit", lambda: H.check_case(c, oracle, workspace=workspace), slices=2) >= 2


def product(A, B, m, n, k, ta=T, tb=N):
    """A (m x k) times the transpose of B (n x k), transposed back: n x m; column-major, op(A) and op(B) stored as ta and tb say"""
    import torch
    out = torch.empty(m * n, device="cuda")
    a, b = (A if ta == T else A.T), (B if tb == N else B.T)
    G.mg_sgemm(C, ta, tb, m, n, k, 1.0, H.to_gpu(np.ascontiguousarray(a)), k if ta == T else m, H.to_gpu(np.ascontiguousarray(b)),
               k if tb == N else n, 0.0, out, m)
    return out.cpu().numpy().reshape(n, m)


@pytest.mark.parametrize("ta,tb", [(T, N), (N, N), (N, T), (T, T)])
@pytest.mark.parametrize("m,n,k", [(256, 128, 64), (131, 257, 75)])
@pytest.mark.parametrize("exponents", ["one", "all"])
def test_a_sum_that_one_product_dominates(ta, tb, m, n, k, exponents):
    """one element that is not zero in each row of op(A) (rows scaled and picked): products of 24-bit elements, nothing else; also with
    elements of every exponent, subnormal ones among them, and products between 2^-100 and 2^87"""
    rng = np.random.default_rng(m + k)
    at = rng.integers(0, k, m)
    A = np.zeros((m, k), np.float32)
    A[np.arange(m), at] = rng.uniform(1, 2, m)
    B = rng.uniform(1, 2, (n, k)).astype(np.float32)
    if exponents == "all":
        ea = np.linspace(-149, 105, k).astype(int)
        eb = np.clip(rng.integers(-100, 85, k) - ea, -120, 105)
        A = np.ldexp(A, ea[None, :]).astype(np.float32)
        B = np.ldexp(B, eb[None, :]).astype(np.float32)
    exact = B.astype(np.float64) @ A.astype(np.float64).T
    outs = []
    assert forced("ssplit", lambda: outs.append(product(A, B, m, n, k, ta, tb))) >= 2
    for got in outs:
        # the last rounding, half a unit; what is added in the last place stays below 2^-6.9 of the product and is rounded seven
        # times, 7 x 2^-24 x 2^-6.9 of it or 1/17 of a unit at most; without a2 b3 + a3 b2 a unit in the last place is reached
        assert np.max(np.abs(got - exact) / np.spacing(exact.astype(np.float32))) <= 0.5 + 1 / 16


@pytest.mark.parametrize("what", ["inf", "nan", "huge", "overflow", "tiny", "subnormal", "bf16_subnormal", "low_bits"])
def test_values_the_parts_cannot_hold(what):
    m, n, k = 200, 150, 300
    rng = np.random.default_rng(5)
    A = rng.uniform(-1, 1, (m, k)).astype(np.float32)
    B = rng.uniform(-1, 1, (n, k)).astype(np.float32)
    if what in ("inf", "nan"):
        A[7, 11] = np.float32(what)
        A[90, 200:210] = np.float32(what)
        B[20, 3] = 0.0
    elif what == "huge":
        A[5, 9] = 3.4e38
        A[130, :] *= 1.0e36                                  # (sums near the end of the range overflow or not by their order)
        B[:, 9] *= 0.01
    elif what == "overflow":
        A *= 1.0e25
        B *= 1.0e25
    elif what == "tiny":
        A *= 1.0e-35
    elif what == "subnormal":
        A[60:70] *= 1.0e-41
        B *= 1.0e20
    elif what == "bf16_subnormal":
        A[60:70] = np.float32(2.0 ** -130)                    # one part holds it
        B *= 1.0e20
    else:
        A = np.ldexp(A, -108).astype(np.float32)             # parts near the end of bf16's range
    runs = {}
    for prefix in ("smfma_64x64", "ssplit"):
        runs[prefix] = []
        assert forced(prefix, lambda: runs[prefix].append(product(A, B, m, n, k))) >= 1
    want = runs["smfma_64x64"][0]
    exact = B.astype(np.float64) @ A.astype(np.float64).T
    size = np.abs(B).astype(np.float64) @ np.abs(A).astype(np.float64).T
    for got in runs["ssplit"]:
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
        ok = np.isfinite(want)
        if what != "overflow":                               # (there the sign is that of whichever partial sum overflows first)
            assert np.array_equal(np.sign(got[~ok & ~np.isnan(want)]), np.sign(want[~ok & ~np.isnan(want)]))
        # k + 1 roundings of sums no larger than `size`, and of subnormals
        with np.errstate(invalid="ignore"):
            assert np.all(np.abs(got - exact)[ok] <= (k + 1) * (2.0 ** -24 * size[ok] + 2.0 ** -149))
        # (that bound is far from what random signs give.  Elements without their last eight bits are off by 2^-19 rms, these sums too: four
        # times what the FP32 pipes' roundings amount to)
        if what in ("tiny", "low_bits", "subnormal", "bf16_subnormal"):
            rows = slice(60, 70) if what.endswith("subnormal") else slice(None)
            off = [np.linalg.norm((x - exact)[:, rows]) / np.linalg.norm(exact[:, rows]) for x in (got, want)]
            assert off[0] <= off[1]


@pytest.mark.parametrize("k", [32, 48, 100, 257, 1024, 4096])
@pytest.mark.parametrize("spread", ["uniform", "wide"])
def test_no_less_precise_than_the_fp32_pipes(k, spread):
    m, n = 256, 256
    rng = np.random.default_rng(k)
    A = rng.uniform(-1, 1, (m, k)).astype(np.float32)
    B = rng.uniform(-1, 1, (n, k)).astype(np.float32)
    if spread == "wide":                                      # magnitudes over forty binades
        A *= np.exp2(rng.integers(-20, 21, (m, k))).astype(np.float32)
        B *= np.exp2(rng.integers(-20, 21, (n, k))).astype(np.float32)
    exact = B.astype(np.float64) @ A.astype(np.float64).T
    for ta, tb in ((T, N), (N, N), (N, T), (T, T)):
        error = {}
        for prefix in ("smfma_64x64", "ssplit"):
            outs = []
            assert forced(prefix, lambda: outs.append(product(A, B, m, n, k, ta, tb))) >= 1
            error[prefix] = max(np.linalg.norm(o - exact) / np.linalg.norm(exact) for o in outs)
        # (where a few products dominate the sum, both are the rounding of those: half a unit in the last place)
        assert error["ssplit"] <= (error["smfma_64x64"] if spread == "uniform" else max(error["smfma_64x64"], 2.0 ** -24))


def call_time(A, B, n, k):
    """microseconds of one n x n x k product, of several in a row"""
    import torch
    out = torch.empty(n * n, device="cuda")
    times = []
    for _ in range(6):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        for _ in range(10):
            G.mg_sgemm(C, T, N, n, n, k, 1.0, A, k, B, k, 0.0, out, n)
        end.record()
        end.synchronize()
        times.append(begin.elapsed_time(end) * 100)
    return sorted(times[1:])[2]


def test_time_does_not_depend_on_small_elements():
    """elements below 2^-110 are products like others (a tile with one of them used to be computed twice: 1.8 times), and NaN ends the
    sum on the bf16 pipes early (2.3 times; now 1.4, the FP32 pipes' share)"""
    import torch
    n, k = 2048, 8192
    A, B = (torch.empty(n, k, device="cuda").uniform_(-1, 1) for _ in range(2))
    assert "ssplit" in G.mg_kernel_name(G.mg_query_selected(G.MG_F32, C, T, N, n, n, k, k, k, n)["kernel_id"])
    usual = call_time(A, B, n, k)
    some = A.clone()
    some[:, 17] = 1.0e-36
    assert call_time(some, B, n, k) < 1.25 * usual
    assert call_time(A * 1.0e-41, B, n, k) < 1.25 * usual
    some[:, 17] = float("nan")
    assert call_time(some, B, n, k) < 1.8 * usual
