"""Batched instances held whole in LDS (csrc/batched_lines.hip): pieces that end beyond a line, a matrix or a column of C, the masked end of the
sum, every operand order, work-groups that walk over many instances, against the CPU oracle, bit for bit on integers."""
import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, R, N, T = W.COL_MAJOR, W.ROW_MAJOR, W.NO_TRANS, W.TRANS


def lines_kernels(dtype):
    code = G.MG_F32 if dtype == "f32" else G.MG_F16
    return [t for t in G.kernel_table() if "batched_lines" in t["name"] and t["dtype"] == code]


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("layout,ta,tb", [(C, N, N), (C, T, N), (C, N, T), (C, T, T), (R, N, N)])
@pytest.mark.parametrize("shape,forms", [((8, 8, 1, 9, 0), 3), ((16, 16, 16, 5, 0), 3), ((3, 17, 9, 7, 2), 3), ((33, 9, 40, 6, 1), 2), ((31, 35, 15, 9, 0), 2),
                                         ((13, 103, 8, 5, 0), 2), ((64, 48, 33, 4, 3), 1), ((68, 68, 68, 3, 3), 1), ((71, 50, 47, 4, 0), 1), ((9, 8, 70, 1100, 1), 1)])
def test_pieces_and_edges_are_exact(oracle, dtype, layout, ta, tb, shape, forms):
    m, n, k, batch, pad = shape
    bc = W.batched_case(m, n, k, batch, case=m + 3 * n + 7 * k, layout=layout, ta=ta, tb=tb, integer=True, dtype=dtype,
                        shuffle_offsets=True, lda=W.tight_ld(layout, ta, m, k) + pad, ldb=W.tight_ld(layout, tb, k, n) + 2 * pad,
                        ldc=W.tight_ld(layout, N, m, n) + pad)
    bc.alphas[1] = 0.0                                           # A and B must not be used
    bc.A[bc.a_off[1]: bc.a_off[1] + W.storage_len(layout, ta, m, k, bc.lda)] = float("nan")
    bc.betas[2] = 0.0
    ran = 0
    try:
        for t in lines_kernels(dtype):
            G.mg_override_batched_config(t["kernel_id"])
            try:
                H.check_batched(bc, oracle, exact=True)
                ran += 1
            except G.MgError as e:
                assert e.status == -11                           # another operand order, or too large for a team
    finally:
        G.mg_clear_override()
    assert ran >= forms
    H.check_batched(bc, oracle, exact=True)


@pytest.mark.parametrize("dtype,m,n,k", [("f16", 20, 17, 13), ("f32", 18, 33, 9), ("f16", 70, 37, 21)])
def test_a_walk_over_many_instances(dtype, m, n, k):
    """more instances than the launch has work-groups; one in seven is not finite, which what it leaves in LDS must not pass on"""
    import torch
    batch, kind = 20011, torch.float32 if dtype == "f32" else torch.float16
    gen = torch.Generator(device="cuda").manual_seed(k)
    draw = lambda *shape: torch.randint(-3, 4, shape, device="cuda", generator=gen, dtype=torch.int8).to(kind)      # noqa: E731
    A, B, old = draw(batch, k, m), draw(batch, n, k), draw(batch, n, m)                                              # column-major instances
    A[::7] = float("nan")
    B[3::7] = float("inf")
    want = torch.zeros(batch, n, m, device="cuda")
    for l in range(k):
        want += B[:, :, l:l + 1].float() * A[:, l:l + 1, :].float()
    want = (2.0 * want - old.float()).to(kind)
    finite = torch.ones(batch, dtype=torch.bool, device="cuda")
    finite[::7] = finite[3::7] = False
    ran = 0
    for t in lines_kernels(dtype):
        if not t["name"].endswith("_mk"):
            continue
        out = old.clone()
        G.mg_override_batched_config(t["kernel_id"])
        try:
            (G.mg_sgemm_strided_batched if dtype == "f32" else G.mg_hgemm_strided_batched)(C, N, N, m, n, k, 2.0, A, m, m * k, B, k, k * n, -1.0, out, m,
                                                                                            m * n, batch)
        except G.MgError as e:
            assert e.status == -11
            continue
        finally:
            G.mg_clear_override()
        ran += 1
        assert torch.equal(out[finite], want[finite])
        assert not torch.isfinite(out[::7]).any()
    assert ran >= 2


def test_what_the_kernels_do_not_take():
    """a matrix of less than 16 bytes, and one that LDS does not hold, run on the other kernels as before"""
    for dtype, m, n, k in (("f16", 1, 40, 5), ("f32", 200, 200, 200)):
        bc = W.batched_case(m, n, k, 4, case=1, layout=C, ta=N, tb=N, integer=True, dtype=dtype)
        for t in lines_kernels(dtype):
            G.mg_override_batched_config(t["kernel_id"])
            try:
                with pytest.raises(G.MgError) as e:
                    H.check_batched(bc, None, exact=True)
                assert e.value.status == -11
            finally:
                G.mg_clear_override()
