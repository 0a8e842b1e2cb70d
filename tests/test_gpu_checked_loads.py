"""FP16 products whose rows start at odd elements: whole K-tiles without checks, against the oracle, where pieces and rows end at
every remainder (a piece of eight rows that straddles the matrix's last one runs into the next line, and the last line has none)."""
import numpy as np
import pytest

from oracle import gemm_oracle
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu
TILES = ("hmfma_64x64x64_w2x2", "hmfma_128x64x64_w2x2", "hmfma_128x128x64_w2x2", "hmfma_256x128x64_w2x2", "hmfma_256x256x64_w2x4")


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("ta,tb,order", [(W.NO_TRANS, W.NO_TRANS, "mk"), (W.NO_TRANS, W.TRANS, "mn"), (W.TRANS, W.NO_TRANS, "kk"),
                                         (W.TRANS, W.TRANS, "kn")])
def test_every_tile(tile, ta, tb, order):
    kernel = G.kernel_id(f"{tile}_{order}_edge")
    # (rows below a piece, one piece, remainders 1 and 7 of a piece; sums that end with, before and behind a K-tile; sums of
    # 1 to 6 K-tiles, whole ones among them, where the last line must not be run over)
    for case, (m, n, k) in enumerate(((3, 5, 128), (8, 9, 64), (65, 71, 129), (129, 263, 192), (257, 255, 256), (131, 137, 321), (33, 47, 447),
                                      (64, 128, 385))):
        for split in (1, 2):
            G.mg_override_config(kernel, split)
            try:
                H.check_case(W.hgemm_case(m, n, k, case=60 + case, ta=ta, tb=tb, beta=0.5), gemm_oracle)
            except G.MgError:
                assert split == 2 and k <= 64, "only a sum of one K-tile has no second slice"
            finally:
                G.mg_clear_override()


def test_buffers_that_end_with_the_matrix():
    """no row padding and NaN behind the last element: nothing behind the matrix reaches the result"""
    import torch
    rng = np.random.default_rng(5)
    for ta, tb in ((G.MG_NO_TRANS, G.MG_TRANS), (G.MG_TRANS, G.MG_NO_TRANS)):
        for m, n, k in ((129, 67, 128), (71, 131, 192), (65, 65, 127)):
            a, b = rng.standard_normal((k, m)).astype(np.float16), rng.standard_normal((k, n)).astype(np.float16)     # op(A)^T, op(B)
            ref = a.astype(np.float64).T @ b.astype(np.float64)
            hold = []
            for x, along_rows in ((a, ta == G.MG_NO_TRANS), (b, tb == G.MG_TRANS)):
                flat = (x if along_rows else x.T).ravel()
                hold.append(torch.from_numpy(np.concatenate([flat, np.full(4096, np.nan, np.float16)])).cuda())
            c = torch.empty(m * n, dtype=torch.float16, device="cuda")
            G.mg_hgemm(G.MG_COL_MAJOR, ta, tb, m, n, k, 1.0, hold[0], m if ta == G.MG_NO_TRANS else k, hold[1],
                       k if tb == G.MG_NO_TRANS else n, 0.0, c, m)
            got = c.cpu().numpy().reshape(n, m).T.astype(np.float64)
            # one rounding to FP16 of a sum kept in FP32: half an ulp of values below 2^7, and k FP32 roundings
            assert np.max(np.abs(got - ref)) <= 2.0 ** -5 + k * 2.0 ** -24 * 64
