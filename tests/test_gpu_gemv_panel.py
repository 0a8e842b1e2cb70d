"""The matrix-vector panel kernels (csrc/gemv.hip): edges of the runs of outputs, of the rounds of loads and of the slices, odd leading
dimensions and increments, against the CPU oracle, bit for bit on integers."""
import numpy as np
import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, R, N, T = W.COL_MAJOR, W.ROW_MAJOR, W.NO_TRANS, W.TRANS


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("layout,trans", [(C, N), (R, T)])
@pytest.mark.parametrize("outputs,length,pad", [(1, 5, 0), (7, 63, 1), (16, 64, 0), (33, 511, 3), (63, 513, 0), (129, 2047, 1), (250, 2561, 5),
                                                (2050, 130, 2), (4099, 40, 0), (33001, 17, 2), (65535, 130, 0)])
def test_panel_edges_are_exact(oracle, dtype, layout, trans, outputs, length, pad):
    m, n = (outputs, length) if trans == N else (length, outputs)
    case = W.gemv_case(dtype, layout, trans, m, n, incx=1 + pad % 2, incy=1 + pad % 3, alpha=2.0, beta=-1.0, integer=True, pad=pad,
                       case=outputs + length)
    try:
        for t in G.kernel_table():
            if "gemv_panel" in t["name"] and t["name"].endswith(dtype):
                for slices in (1, 3):
                    if slices > length:
                        continue
                    G.mg_override_config(t["kernel_id"], slices)
                    H.check_gemv(case, oracle)
    finally:
        G.mg_clear_override()
    H.check_gemv(case, oracle)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("m,n", [(4096, 2561), (2048, 4224), (2047, 4225), (4160, 4100), (512, 12000)])
@pytest.mark.parametrize("workspace", ["auto", None])
def test_both_sides_of_the_selection(oracle, dtype, m, n, workspace):
    case = W.gemv_case(dtype, C, N, m, n, alpha=0.5, beta=2.0, case=m + n)
    H.check_gemv(case, oracle, workspace=workspace)


def test_infinities_stay_in_their_row(oracle):
    """a tail of the sum is no product with zero: Inf in A stays Inf, and only in its own output"""
    import torch
    m, n = 70, 2600
    A = torch.rand(m * n, device="cuda")
    A[5 + (n - 1) * m] = float("inf")
    x, y = torch.rand(n, device="cuda") + 0.5, torch.zeros(m, device="cuda")
    ws = torch.empty(max(1, G.mg_gemv_workspace_bytes(G.MG_F32, C, N, m, n, m)), dtype=torch.uint8, device="cuda")
    G.mg_sgemv(C, N, m, n, 1.0, A, m, x, 1, 0.0, y, 1, ws)
    out = y.cpu().numpy()
    assert np.isposinf(out[5]) and np.isfinite(np.delete(out, 5)).all()


@pytest.mark.parametrize("dtype,outputs,length,ld", [("f32", 64, 400000, 1024), ("f32", 128, 200001, 1024), ("f32", 2048, 16384, 2048),
                                                     ("f16", 128, 390001, 2048), ("f16", 4096, 16384, 4096)])
def test_sums_sliced_over_a_streamed_matrix(dtype, outputs, length, ld):
    """more than 96 MB with columns a multiple of 4 KB apart, up to as many slices as there are; integers, exact but for the rounding
    of the result"""
    import torch
    f32 = dtype == "f32"
    kind = torch.float32 if f32 else torch.float16
    gen = torch.Generator(device="cuda").manual_seed(outputs)
    A = torch.full((length, ld), float("nan"), device="cuda", dtype=kind)
    A[:, :outputs] = torch.randint(-3, 4, (length, outputs), device="cuda", generator=gen, dtype=torch.int8).to(kind)
    x = torch.randint(-3, 4, (length,), device="cuda", generator=gen).to(kind)
    y = torch.randint(-3, 4, (outputs,), device="cuda", generator=gen).to(kind)
    want = 2.0 * torch.mv(A[:, :outputs].t().double(), x.double()) - y.double()
    ws = torch.empty(G.mg_gemv_workspace_bytes(G.MG_F32 if f32 else G.MG_F16, C, N, outputs, length, ld), dtype=torch.uint8, device="cuda")
    (G.mg_sgemv if f32 else G.mg_hgemv)(C, N, outputs, length, 2.0, A, ld, x, 1, -1.0, y, 1, ws)
    assert torch.equal(y, want.to(kind))


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("outputs", [1, 3, 4, 5, 7, 8, 9, 257, 511, 513, 519])
@pytest.mark.parametrize("length", [1, 40, 700])
def test_where_the_outputs_end(oracle, dtype, outputs, length):
    """inside the first run, with a run, inside a later one and inside the first run of a work-group, on every kernel along the outputs"""
    case = W.gemv_case(dtype, C, N, outputs, length, incy=2, alpha=2.0, beta=-1.0, integer=True, pad=1, case=outputs + length)
    ran = 0
    try:
        for t in G.kernel_table():
            if t["name"].startswith(("gemv_panel", "gemv_axpy")) and t["name"].endswith(dtype):
                G.mg_override_config(t["kernel_id"], 1)
                H.check_gemv(case, oracle)
                ran += 1
    finally:
        G.mg_clear_override()
    assert ran >= 4
