"""NCHW source gradient of more channels than a grid has in z: the flipped
filter copy then goes through the KRSC filter."""
import pytest
import torch

import oracle
from paper_1603_07846_amd import singa
from paper_1603_07846_amd import workloads as wl
from _helpers import TOL, dev_to_nchw, kcrs_to_dev, nchw_to_dev, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("C", [65535, 65544])
def test_source_gradient_of_many_channels(C, dt):
    N, H, K = 2, 2, 8
    w = wl.random_array((K, C, 1, 1), 600, "normal", 0.1, dt)
    dy = wl.random_array((N, K, H, H), 601, "normal", 1.0, dt)
    dx = singa.conv_bwd_data(nchw_to_dev(dy, dt, "NCHW"), kcrs_to_dev(w, dt, "NCHW"), (N, C, H, H), layout="NCHW")
    torch.cuda.synchronize()
    assert rel_l2(dev_to_nchw(dx, "NCHW"), oracle.conv_bwd_data(dy, w, (N, C, H, H), pad=0, stride=1)) <= TOL[dt]
