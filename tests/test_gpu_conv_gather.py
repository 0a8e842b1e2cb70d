"""Convolutions in one launch from a band of the image in LDS (csrc/conv_gather.hip): output positions and filters beside the 32 x 32 blocks, every
width of the band's pieces, sums that end inside a K-step, bands in several chunks of channels, padding, stride and dilation, against the CPU
oracle, bit for bit on integers; the calls that keep their former routes."""
import pytest

import helpers as H
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def CO():
    from oracle import conv_oracle
    return conv_oracle


def kernels(dtype, *geo, beta=0.0):
    """names of the kernels that one call launches"""
    import torch
    from torch.profiler import ProfilerActivity, profile
    case = W.conv_case(dtype, *geo, beta=beta)
    im, w, out = H.to_gpu(case.im), H.to_gpu(case.weights), H.to_gpu(case.out)
    code = G.MG_F32 if dtype == "f32" else G.MG_F16
    args = (case.channels, case.height, case.width, case.kernel, case.pad, case.stride, case.dilation)
    ws = torch.empty(max(256, G.mg_conv2d_workspace_bytes(code, *args, case.filters)), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as record:
        (G.mg_sconv2d if dtype == "f32" else G.mg_hconv2d)(*args, case.filters, case.alpha, im, w, case.beta, out, ws)
        torch.cuda.synchronize()
    return [e.name for e in record.events() if "mg::" in e.name or "_ZN2mg" in e.name]


GEO = [
    # channels, height, width, kernel, pad, stride, dilation, filters
    (16, 8, 8, (3, 3), (1, 1), (1, 1), (1, 1), 32),         # 64 positions; pieces of eight (FP16), four (FP32)
    (16, 5, 12, (3, 3), (1, 1), (1, 1), (1, 1), 33),        # 60 positions, 33 filters; pieces of four
    (7, 9, 14, (3, 3), (1, 1), (2, 2), (1, 1), 31),         # 35 positions, 63 terms; pieces of two, stride
    (3, 7, 7, (7, 7), (3, 3), (2, 2), (1, 1), 5),           # single elements, wide padding, 147 terms
    (1, 1, 1, (1, 1), (1, 1), (1, 1), (1, 1), 1),           # one term, nine positions, eight of them padding
    (2, 33, 3, (3, 1), (1, 0), (1, 1), (2, 1), 40),         # three positions a row: the band of a block is a dozen rows; dilation down
    (5, 6, 40, (2, 5), (0, 4), (3, 2), (1, 2), 64),         # dilation across, padding wider than the filter's half
    (65, 7, 7, (3, 3), (1, 1), (1, 1), (1, 1), 32),         # 585 terms: the last K-step is partial
    (9, 2, 136, (3, 3), (1, 1), (1, 1), (1, 1), 16),        # most blocks begin and end inside a row
    (182, 19, 8, (1, 1), (2, 1), (4, 4), (1, 1), 33),       # the band comes in two chunks of channels, the second one smaller
]


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("geo", GEO)
def test_blocks_bands_and_sums(CO, dtype, geo):
    for integer in (True, False):
        case = W.conv_case(dtype, *geo, alpha=1.0 if integer else 0.75, beta=1.0 if integer else -0.5, case=11, integer=integer)
        H.check_conv(case, CO, "auto")
    ran = kernels(dtype, *geo)
    # (182 channels in FP32: the rows outside the image are most of the band, and the unfold route is the better one; test_any_layer_on_this_kernel has it)
    if (dtype, geo[0]) != ("f32", 182):
        assert len(ran) == 1 and "conv_gather" in ran[0], ran


def odd_layers():
    """small layers of any geometry: about a third of them with one to three positions, filters or channels"""
    import random
    rng = random.Random(6)
    layers = []
    while len(layers) < 120:
        few = lambda most: rng.randint(1, 3) if rng.random() < 0.3 else rng.randint(1, most)       # noqa: E731
        kernel, dilation = (rng.choice((1, 2, 3, 5, 7)), rng.choice((1, 3, 4))), (rng.choice((1, 1, 2, 3)), rng.choice((1, 1, 2, 3)))
        pad, stride = (rng.randint(0, 4), rng.randint(0, 9)), (rng.randint(1, 4), rng.randint(1, 4))
        channels, height, width, filters = few(90), few(40), few(70), few(80)
        extents = [(size + 2 * p - d * (x - 1) - 1) // s + 1 for size, x, p, s, d in zip((height, width), kernel, pad, stride, dilation)]
        if min(extents) >= 1 and channels * kernel[0] * kernel[1] * extents[0] * extents[1] * filters < 4e7:
            layers.append((channels, height, width, kernel, pad, stride, dilation, filters))
    return layers


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("geo", GEO + odd_layers())
def test_any_layer_on_this_kernel(CO, dtype, geo):
    """not the library's choice: every layer that the kernel takes"""
    import numpy as np
    case = W.conv_case(dtype, *geo, alpha=1.0, beta=1.0 if geo[0] % 2 else 0.0, case=13, integer=True)
    if case.beta == 0.0:
        case.out[:] = np.nan
    want, _ = CO.conv2d(dtype, *H.conv_geometry(case), case.filters, case.alpha, case.im, case.weights, case.beta, case.out)
    im, weights, out = H.to_gpu(case.im), H.to_gpu(case.weights), H.to_gpu(case.out)
    G.mg_probe_conv_gather(G.MG_F32 if dtype == "f32" else G.MG_F16, *H.conv_geometry(case), case.filters, case.alpha, im, weights, case.beta, out)
    assert np.array_equal(out.cpu().numpy().astype(np.float64), want)


def test_layers_whose_rows_do_not_fit_are_refused():
    """sixteen channels of a band of 7 rows of 1000 elements in FP32"""
    import torch
    x = torch.zeros(64 * 7 * 1000, device="cuda")
    assert G.mg_probe_conv_gather(G.MG_F32, 64, 7, 1000, (7, 7), (3, 3), (1, 1), (1, 1), 1, 1.0, x, x, 0.0, x.clone(), check=False) == -11
    assert G.mg_probe_conv_gather(G.MG_F32, 64, 7, 100, (3, 3), (1, 1), (1, 1), (1, 1), 1, 0.0, x, x, 0.0, x.clone(), check=False) == -11
    assert G.mg_probe_conv_gather(7, 64, 7, 100, (3, 3), (1, 1), (1, 1), (1, 1), 1, 1.0, x, x, 0.0, x.clone(), check=False) == -11


def test_two_chunks_of_channels_f32(CO):
    """64 channels of the band, then 36, 2500 terms"""
    geo = (100, 56, 56, (5, 5), (2, 2), (1, 1), (1, 1), 33)
    for integer in (True, False):
        H.check_conv(W.conv_case("f32", *geo, alpha=1.0 if integer else 0.75, beta=1.0 if integer else -0.5, case=11, integer=integer), CO, "auto")
    ran = kernels("f32", *geo)
    assert len(ran) == 1 and "conv_gather" in ran[0], ran


def test_infinite_pixels_stay_where_they_are(CO):
    """an infinite pixel reaches the outputs that see it, no other: nothing multiplies zeros from outside the sum with it"""
    import numpy as np
    case = W.conv_case("f32", 3, 9, 9, (3, 3), (1, 1), (1, 1), (1, 1), 4, beta=0.0, case=2)
    case.im.reshape(3, 9, 9)[1, 4, 4] = np.inf
    out = H.run_conv(case, "auto").reshape(4, 9, 9)
    seen = np.zeros((9, 9), bool)
    seen[3:6, 3:6] = True
    assert np.isinf(out[:, seen]).all() and np.isfinite(out[:, ~seen]).all()


@pytest.mark.parametrize("dtype,geo", [("f16", (64, 93, 93, (3, 3), (1, 1), (1, 1), (1, 1), 261)), ("f32", (16, 63, 63, (3, 3), (1, 1), (1, 1), (1, 1), 448)),
                                       ("f16", (512, 7, 7, (3, 3), (1, 1), (1, 1), (1, 1), 512)),
                                       ("f16", (447, 98, 98, (3, 3), (1, 1), (1, 1), (1, 1), 32)), ("f32", (306, 84, 84, (3, 3), (1, 1), (1, 1), (1, 1), 104)),
                                       ("f32", (64, 85, 85, (7, 7), (3, 3), (1, 1), (1, 1), 80)), ("f32", (16, 106, 106, (3, 3), (1, 1), (1, 1), (1, 1), 115))])
def test_larger_layers_keep_the_unfold_route(dtype, geo):
    """22 / 65, 15 / 21, 17.6 / 20.8, 62 / 114, 80 / 126, 87 / 102 and 17.5 / 20.1 us"""
    assert any("im2col" in name for name in kernels(dtype, *geo))


@pytest.mark.parametrize("geo", [(480, 64, 64, (5, 5), (2, 2), (2, 2), (1, 1), 249), (185, 43, 43, (7, 7), (3, 3), (1, 1), (1, 1), 113),
                                 (42, 198, 198, (3, 3), (1, 1), (1, 1), (1, 1), 29)])
def test_layers_of_many_loads_and_little_gain_keep_the_unfold_route(geo):
    """FP32, bands in several chunks and grids of several turns: 80 / 96, 66 / 74 and 44 / 50 us"""
    assert any("im2col" in name for name in kernels("f32", *geo))


def test_error_of_an_evenly_shared_sum():
    """FP32, 200 terms: an error against 64 bits of at most that of 25 K-steps of eight terms dealt to the eight wavefronts in turn, term by term.

    3 % on top for another order of the terms.  Shares rounded up to four K-steps, on seven wavefronts, have 1.06 times this error, equal ones
    0.99 times."""
    import numpy as np
    import torch
    channels, size, filters, k = 8, 30, 100, 200
    out = size - 4
    rng = np.random.default_rng(5)
    im = (rng.random((channels, size, size)) * 2 - 1).astype(np.float32)
    weights = (rng.random((filters, k)) * 2 - 1).astype(np.float32)
    windows = np.lib.stride_tricks.sliding_window_view(im, (5, 5), axis=(1, 2))
    columns = windows.transpose(0, 3, 4, 1, 2).reshape(k, out * out)
    exact = weights.astype(np.float64) @ columns.astype(np.float64)
    total = np.zeros_like(exact, dtype=np.float32)
    for wave in range(8):
        s = np.zeros_like(total)
        for l in range(k):
            if l // 8 % 8 == wave:
                s = (s.astype(np.float64) + np.outer(weights[:, l].astype(np.float64), columns[l].astype(np.float64))).astype(np.float32)
        total += s
    assert any("conv_gather" in n for n in kernels("f32", channels, size, size, (5, 5), (0, 0), (1, 1), (1, 1), filters))
    geometry = (channels, size, size, (5, 5), (0, 0), (1, 1), (1, 1))
    ws = torch.empty(max(256, G.mg_conv2d_workspace_bytes(G.MG_F32, *geometry, filters)), dtype=torch.uint8, device="cuda")
    got = torch.zeros(filters, out * out, device="cuda")
    G.mg_sconv2d(*geometry, filters, 1.0, torch.from_numpy(im).cuda(), torch.from_numpy(weights).cuda(), 0.0, got, ws)
    error = lambda x: np.linalg.norm(x.astype(np.float64) - exact) / np.linalg.norm(exact)
    assert error(got.cpu().numpy()) <= 1.03 * error(total)


@pytest.mark.parametrize("channels,size,kernel,filters", [(64, 28, 3, 32), (153, 51, 3, 37), (100, 56, 5, 33)])
def test_error_of_a_long_sum(channels, size, kernel, filters):
    """FP32, 576 to 2500 terms: an error against 64 bits of at most that of sixteen equal parts of the sum, added up term by term.

    5 % on top for another order of the terms.  Sixteen is what the unfold route cuts long sums into; eight parts have 1.21 to 1.36 times this error."""
    import numpy as np
    import torch
    pad, k = kernel // 2, channels * kernel * kernel
    rng = np.random.default_rng(5)
    im = (rng.random((channels, size, size)) * 2 - 1).astype(np.float32)
    weights = (rng.random((filters, k)) * 2 - 1).astype(np.float32)
    windows = np.lib.stride_tricks.sliding_window_view(np.pad(im, ((0, 0), (pad, pad), (pad, pad))), (kernel, kernel), axis=(1, 2))
    columns = windows.transpose(0, 3, 4, 1, 2).reshape(k, size * size)
    exact = weights.astype(np.float64) @ columns.astype(np.float64)
    total = np.zeros_like(exact, dtype=np.float32)
    for part in np.array_split(np.arange(k), 16):
        s = np.zeros_like(total)
        for l in part:
            s = (s.astype(np.float64) + np.outer(weights[:, l].astype(np.float64), columns[l].astype(np.float64))).astype(np.float32)
        total += s
    geo = (channels, size, size, (kernel, kernel), (pad, pad), (1, 1), (1, 1))
    assert any("conv_gather" in n for n in kernels("f32", *geo, filters))
    ws = torch.empty(max(256, G.mg_conv2d_workspace_bytes(G.MG_F32, *geo, filters)), dtype=torch.uint8, device="cuda")
    got = torch.zeros(filters, size * size, device="cuda")
    G.mg_sconv2d(*geo, filters, 1.0, torch.from_numpy(im).cuda(), torch.from_numpy(weights).cuda(), 0.0, got, ws)
    error = lambda x: np.linalg.norm(x.astype(np.float64) - exact) / np.linalg.norm(exact)
    assert error(got.cpu().numpy()) <= 1.05 * error(total)


@pytest.mark.parametrize("dtype,channels,size,kernel,stride,filters,kernels_in_order", [
    ("f32", 64, 140, 3, 1, 22, ["conv_gather"]),                                                             # 40.7 / 25.2
    ("f16", 16, 111, 3, 1, 13, ["conv_gather"]),                                                             # a thin product 31.4 / 8.0
    ("f16", 7, 116, 3, 1, 32, ["mfma"]), ("f16", 64, 65, 1, 2, 35, ["mfma"]),      # 8.5 / 6.1, 8.0 / 5.9
    ("f32", 64, 45, 1, 2, 28, ["im2col", "tiny"]), ("f16", 3, 44, 7, 1, 194, ["im2col", "kernel"])])           # 8.4 / 6.4, 11.0 / 8.8
def test_routes(dtype, channels, size, kernel, stride, filters, kernels_in_order):
    """us on another route / on this"""
    pair = lambda v: (v, v)                     # noqa: E731
    ran = kernels(dtype, channels, size, size, pair(kernel), pair(kernel // 2), pair(stride), (1, 1), filters)
    assert len(ran) == len(kernels_in_order) and all(part in name for part, name in zip(kernels_in_order, ran)), ran


def test_thin_products_behind_the_unfold_pass_with_any_workspace():
    """FP32, 1600 terms, 5 filters: with room for slices, which so thin a product does not take, the sum is shared all the same (an error of 1.5e-7, one chain 7.1e-7)"""
    import torch
    geo, filters = (64, 97, 97, (5, 5), (2, 2), (2, 2), (1, 1)), 5
    im, w = torch.rand(64, 97, 97, device="cuda") * 2 - 1, torch.rand(filters, 1600, device="cuda") * 2 - 1
    exact = torch.from_numpy(w.cpu().double().numpy()) @ torch.nn.functional.unfold(im.cpu().double()[None], 5, padding=2, stride=2)[0]
    got = torch.zeros(filters, 49 * 49, device="cuda")
    G.mg_sconv2d(*geo, filters, 1.0, im, w, 0.0, got, torch.empty(1 << 26, dtype=torch.uint8, device="cuda"))
    assert (got.cpu().double() - exact).norm() <= 3.0e-7 * exact.norm()


def test_first_layer_keeps_the_fused_route():
    """9.2 / 18.3 us"""
    ran = kernels("f16", 3, 224, 224, (7, 7), (3, 3), (2, 2), (1, 1), 64)
    assert not any("conv_gather" in name for name in ran), ran
