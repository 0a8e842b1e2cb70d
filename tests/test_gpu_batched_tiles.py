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
    try:
        for t in G.kernel_table():                               # every tile that takes the shape, then the selection
            if "batched_tile" in t["name"] and t["dtype"] == (G.MG_F32 if dtype == "f32" else G.MG_F16):
                G.mg_override_batched_config(t["kernel_id"])
                try:
                    H.check_batched(bc, oracle, exact=True)
                except G.MgError as e:
                    assert e.status == -11                       # another operand order, or too large for one wavefront
    finally:
        G.mg_clear_override()
    H.check_batched(bc, oracle, exact=True)
