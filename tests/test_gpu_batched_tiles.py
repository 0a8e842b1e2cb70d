"""Batched instances beyond the one-wavefront kernels (csrc/batched_tile.hip): edges of the tiles, of the chunks of k and of the
16-byte pieces, every operand order, against the CPU oracle, bit for bit on integers."""
import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, R, N, T = W.COL_MAJOR, W.ROW_MAJOR, W.NO_TRANS, W.TRANS


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("layout,ta,tb", [(C, N, N), (C, T, N), (C, N, T), (C, T, T), (R, N, N)])
@pytest.mark.parametrize("shape", [(33, 1, 1, 9, 0), (1, 33, 65, 8, 1), (32, 32, 33, 13, 0), (17, 30, 130, 7, 3), (64, 64, 64, 5, 1),
                                   (65, 63, 31, 4, 0), (66, 129, 97, 3, 2), (128, 128, 64, 17, 0), (200, 7, 16, 3, 5)])
def test_tile_edges_are_exact(oracle, dtype, layout, ta, tb, shape):
    m, n, k, batch, pad = shape
    bc = W.batched_case(m, n, k, batch, case=m + 3 * n + 7 * k, layout=layout, ta=ta, tb=tb, integer=True, dtype=dtype,
                        shuffle_offsets=True, lda=W.tight_ld(layout, ta, m, k) + pad, ldb=W.tight_ld(layout, tb, k, n) + 2 * pad,
                        ldc=W.tight_ld(layout, N, m, n) + pad)
    bc.alphas[1] = 0.0                                           # A and B must not be used
    bc.A[bc.a_off[1]: bc.a_off[1] + W.storage_len(layout, ta, m, k, bc.lda)] = float("nan")
    bc.betas[2] = 0.0
    ran = 0
    try:
        for t in G.kernel_table():                               # every tile that takes the shape, then the selection
            if "batched_tile" in t["name"] and t["dtype"] == (G.MG_F32 if dtype == "f32" else G.MG_F16):
                G.mg_override_batched_config(t["kernel_id"])
                try:
                    H.check_batched(bc, oracle, exact=True)
                    ran += 1
                except G.MgError as e:
                    assert e.status == -11                       # another operand order, or too large for one wavefront
    finally:
        G.mg_clear_override()
    assert ran == 2 + (m <= 32 and n <= 32)
    H.check_batched(bc, oracle, exact=True)


@pytest.mark.parametrize("dtype,m,n,k,strided", [("f16", 40, 1, 1, True), ("f32", 33, 1, 2, False)])
def test_more_instances_than_one_launch_takes(dtype, m, n, k, strided):
    """2^24 + 1003 instances on kernels with one work-group per instance: every instance has its own operands and scalars (small
    integers, exact in either type)"""
    import torch
    batch, f32 = 2 ** 24 + 1003, dtype == "f32"
    gen = torch.Generator(device="cuda").manual_seed(m)
    draw = lambda *shape: torch.randint(-3, 4, shape, device="cuda", generator=gen, dtype=torch.int8)      # noqa: E731
    kind = torch.float32 if f32 else torch.float16
    A, B, Cm = (draw(batch, x, y).to(kind) for x, y in ((k, m), (n, k), (n, m)))                           # column-major instances
    alphas, betas = draw(batch).float(), draw(batch).float()
    old = Cm.clone()
    if strided:
        (G.mg_sgemm_strided_batched if f32 else G.mg_hgemm_strided_batched)(C, N, N, m, n, k, 2.0, A, m, m * k, B, k, k * n, -1.0,
                                                                            Cm, m, m * n, batch)
        alphas, betas = 2.0, -1.0
    else:
        place = torch.arange(batch, dtype=torch.int64, device="cuda")
        (G.mg_sgemm_batched if f32 else G.mg_hgemm_batched)(C, N, N, m, n, k, alphas, A, place * (m * k), m, B, place * (k * n), k,
                                                            betas, Cm, place * (m * n), m, batch)
        alphas, betas = alphas.view(-1, 1, 1), betas.view(-1, 1, 1)
    want = betas * old
    for l in range(k):
        want += alphas * B[:, :, l:l + 1] * A[:, l:l + 1, :]
    assert torch.equal(Cm, want.to(kind))
