"""Strided FP16 batches on the direct-to-LDS tiles (csrc/batched_dma.hip): instances beside each tile, all operand orders, beta, gaps between instances
and lines, against the CPU oracle, bit for bit on integers; batches whose pieces are off 16 bytes keep their kernels."""
import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu

C, R, N, T = W.COL_MAJOR, W.ROW_MAJOR, W.NO_TRANS, W.TRANS


def run(m, n, k, batch, layout, ta, tb, beta, pad, gap, pad_c=None, gap_c=None, off_c=0, tile=None):
    """(names of the kernels, C of every instance, expected C of every instance); what lies beside the instances is NaN.  pad, gap: elements behind
    a line and an instance, off_c: in front of C; tile: not the library's choice"""
    import numpy as np
    import torch
    from torch.profiler import ProfilerActivity, profile
    rng = np.random.default_rng(m * 131 + n * 17 + k)
    made = []
    pad_c, gap_c = pad if pad_c is None else pad_c, gap if gap_c is None else gap_c
    for rows, cols, pad, gap, off in ((*W.stored_extents(ta, m, k), pad, gap, 0), (*W.stored_extents(tb, k, n), pad, gap, 0), (m, n, pad_c, gap_c, off_c)):
        minor, major = (rows, cols) if layout == C else (cols, rows)
        ld = minor + pad
        stride = ld * major + gap
        buf = np.full(off + stride * batch, np.nan, dtype=np.float16)
        view = np.lib.stride_tricks.as_strided(buf[off:], (batch, major, minor), (2 * stride, 2 * ld, 2))
        view[:] = rng.integers(-2, 3, (batch, major, minor))
        made.append((buf, ld, stride, view.astype(np.float64).transpose(0, 2, 1) if layout == C else view.astype(np.float64)))
    (a, lda, sa, A), (b, ldb, sb, B), (c, ldc, sc, Cm) = made
    want = np.matmul(A.transpose(0, 2, 1) if ta != N else A, B.transpose(0, 2, 1) if tb != N else B) + beta * Cm
    da, db, dc = (torch.from_numpy(x).cuda() for x in (a, b, c))
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as record:
        call = G.mg_hgemm_strided_batched if tile is None else lambda *args: G.mg_probe_hgemm_batched_tile(tile, *args)
        call(layout, ta, tb, m, n, k, 1.0, da, lda, sa, db, ldb, sb, beta, dc[off_c:], ldc, sc, batch)
        torch.cuda.synchronize()
    got = dc.cpu().numpy()
    minor, major = (m, n) if layout == C else (n, m)
    out = np.lib.stride_tricks.as_strided(got[off_c:], (batch, major, minor), (2 * sc, 2 * ldc, 2)).astype(np.float64)
    rest = got.copy()
    np.lib.stride_tricks.as_strided(rest[off_c:], (batch, major, minor), (2 * sc, 2 * ldc, 2))[:] = np.nan
    assert np.isnan(rest).all()                                 # nothing beside the instances was written
    names = [e.name for e in record.events() if "mg::" in e.name or "_ZN2mg" in e.name]
    return names, out.transpose(0, 2, 1) if layout == C else out, want


@pytest.mark.parametrize("layout", [C, R])
@pytest.mark.parametrize("ta,tb", [(N, N), (T, N), (N, T), (T, T)])
@pytest.mark.parametrize("m,n,k,batch,beta,pad,gap,tile", [(128, 128, 64, 9, 0.0, 0, 0, "128, 128"), (136, 120, 72, 3, 1.0, 8, 8, ""), (120, 128, 8, 5, -1.0, 0, 16, "128, 128"),
                                                           (64, 64, 72, 17, 0.0, 8, 0, "64, 64"), (72, 136, 136, 2, 1.0, 0, 8, ""), (40, 56, 192, 3, 1.0, 0, 0, "64, 64")])
def test_instances_beside_a_tile(layout, ta, tb, m, n, k, batch, beta, pad, gap, tile):
    import numpy as np
    names, got, want = run(m, n, k, batch, layout, ta, tb, beta, pad, gap)
    assert len(names) == 1 and f"hbatched_dma_kernel<{tile}" in names[0], names
    assert np.array_equal(got, want)


@pytest.mark.parametrize("m,n,k,pad,gap", [(128, 128, 64, 0, 4), (128, 128, 64, 1, 0), (128, 128, 60, 0, 0), (24, 128, 64, 0, 0)])
def test_others_keep_their_kernels(m, n, k, pad, gap):
    import numpy as np
    names, got, want = run(m, n, k, 5, C, T, N, 0.0, pad, gap)
    assert not any("hbatched_dma" in name for name in names)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("layout", [C, R])
@pytest.mark.parametrize("ta,tb", [(N, N), (T, N), (N, T), (T, T)])
@pytest.mark.parametrize("tile", [0, 1, 2])
@pytest.mark.parametrize("m,n,k,batch,beta,pad_c,gap_c,off_c", [(8, 8, 8, 11, 0.0, 1, 0, 0), (136, 72, 64, 3, 1.0, 3, 5, 1), (64, 128, 200, 2, -1.0, 0, 1, 0), (128, 64, 72, 3, 1.0, 0, 3, 7),
                                                                (200, 264, 16, 2, 1.0, 5, 0, 3), (120, 56, 136, 9, 0.0, 2, 2, 2)])
def test_any_place_of_c(layout, ta, tb, tile, m, n, k, batch, beta, pad_c, gap_c, off_c):
    """every tile on every size: leading dimension, stride and address of C at any element"""
    import numpy as np
    _, got, want = run(m, n, k, batch, layout, ta, tb, beta, 8, 16, pad_c, gap_c, off_c, tile)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("pad_c,gap_c,off_c", [(1, 0, 0), (0, 3, 0), (0, 0, 1), (3, 5, 7)])
def test_the_choice_does_not_depend_on_c(pad_c, gap_c, off_c):
    import numpy as np
    names, got, want = run(128, 120, 64, 9, C, T, N, 1.0, 0, 0, pad_c, gap_c, off_c)
    assert len(names) == 1 and "hbatched_dma_kernel" in names[0], names
    assert np.array_equal(got, want)


def test_what_the_tiles_do_not_take_is_refused():
    import torch
    a = torch.zeros(1 << 16, dtype=torch.float16, device="cuda")
    good = dict(tile=0, m=64, n=64, k=64, alpha=1.0, lda=64, sa=4096, ldb=64, sb=4096, at=a)
    for wrong in (dict(tile=3), dict(tile=-1), dict(alpha=0.0), dict(k=0), dict(k=60), dict(lda=68), dict(sb=4100), dict(at=a[4:])):
        v = {**good, **wrong}
        status = G.mg_probe_hgemm_batched_tile(v["tile"], C, T, N, v["m"], v["n"], v["k"], v["alpha"], v["at"], v["lda"], v["sa"], a, v["ldb"], v["sb"], 0.0,
                                               a[32768:], 64, 4096, 4, check=False)
        assert status == -11, wrong
