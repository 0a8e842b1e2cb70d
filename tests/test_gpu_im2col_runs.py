"""IM2COL with a horizontal stride of one, whose threads in FP16 read two runs of image elements: output rows of just 16 bytes and a little
more, runs that start before the image or end behind it, images smaller than a run; bit-exact against the oracle."""
import numpy as np
import pytest

from oracle import conv_oracle
from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("geo", [
    (1, 1, 2, (1, 3), (0, 4), (1, 1), (1, 1), 1),              # fewer elements than a run
    (3, 5, 4, (3, 3), (1, 1), (1, 1), (1, 1), 1),              # output rows of 4: too short for the runs
    (2, 6, 8, (3, 3), (1, 1), (1, 1), (1, 1), 1),              # ... of 8
    (2, 6, 9, (3, 3), (1, 1), (1, 1), (1, 1), 1),
    (2, 9, 12, (5, 5), (4, 4), (1, 1), (1, 1), 1),             # more padding than the filter needs
    (2, 9, 15, (3, 3), (7, 9), (2, 1), (2, 3), 1),             # padding beyond the image, dilation, vertical stride
    (5, 31, 33, (3, 2), (0, 1), (3, 1), (1, 1), 1),
    (37, 23, 29, (7, 7), (3, 3), (1, 1), (1, 1), 1),
])
def test_runs(dtype, geo):
    import torch
    case = W.conv_case(dtype, *geo, case=4)
    oh, ow = case.out_hw
    total = case.k * oh * ow
    im = H.to_gpu(case.im)
    col = torch.full((total + 64,), -77.0, dtype=im.dtype, device="cuda")
    (G.mg_sim2col if dtype == "f32" else G.mg_him2col)(*H.conv_geometry(case), im, col)
    host = col.cpu().numpy()
    assert np.all(host[total:] == -77.0)
    assert np.array_equal(host[:total].astype(np.float64).reshape(case.k, oh * ow), conv_oracle.im2col(dtype, *H.conv_geometry(case), case.im))
