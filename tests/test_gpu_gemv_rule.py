"""Dense layers of one to three rows on both sides of the line between the
matrix-vector kernel and the tiles: the kernel that runs, and its result."""
import pytest
import torch

import oracle
from paper_1603_07846_amd import singa
from paper_1603_07846_amd import workloads as wl
from _helpers import TOL, dev_to_nchw, kcrs_to_dev, nchw_to_dev, phys, rel_l2

pytestmark = pytest.mark.gpu

# dtype, rows, columns, least taps of the matrix-vector kernel
LINE = [("bf16", 1, 4104, 512), ("bf16", 2, 1024, 128), ("bf16", 2, 1032, 256), ("bf16", 2, 4104, 2048),
        ("bf16", 3, 32, 96), ("bf16", 3, 33, 256), ("bf16", 3, 4096, 512), ("bf16", 3, 4097, 2048),
        ("f32", 2, 4097, 64), ("f32", 3, 4100, 128)]


@pytest.mark.parametrize("side", ["below", "at"])
@pytest.mark.parametrize("dt,N,K,taps", LINE, ids=["-".join(map(str, c)) for c in LINE])
def test_few_rows_kernel(dt, N, K, taps, side):
    vec = 8 if dt == "bf16" else 4
    C = taps if side == "at" else taps - vec
    x = wl.random_array((N, C, 1, 1), 500, "normal", 1.0, dt)
    w = wl.random_array((K, C, 1, 1), 501, "normal", 0.1, dt)
    b = wl.random_array((K,), 502, "normal", 0.1, "f32")
    singa.trace_enable(True)
    y = singa.conv_fwd(nchw_to_dev(x, dt), kcrs_to_dev(w, dt), torch.from_numpy(b).cuda())
    torch.cuda.synchronize()
    names = [r[0] for r in singa.trace_records()]
    singa.trace_enable(False)
    assert (names == ["conv_fwd_kernel<%s,gemv,0>" % dt]) == (side == "at"), names
    assert rel_l2(dev_to_nchw(y), oracle.conv_fwd(x, w, b, pad=0, stride=1)) <= TOL[dt]


def test_source_gradient_of_a_wide_layer_with_few_filters():
    """fp32, three rows, 16 filters over 9216 inputs: a reduction of 16 terms,
    on tiles (the matrix-vector kernel took 13.6 us for it, the tiles 6.7)."""
    N, C, K = 3, 9216, 16
    w = wl.random_array((K, C, 1, 1), 503, "normal", 0.1, "f32")
    dy = wl.random_array((N, K, 1, 1), 504, "normal", 1.0, "f32")
    singa.trace_enable(True)
    dx = singa.conv_bwd_data(nchw_to_dev(dy), kcrs_to_dev(w), phys((N, C, 1, 1)))
    torch.cuda.synchronize()
    names = [r[0] for r in singa.trace_records()]
    singa.trace_enable(False)
    assert not any("gemv" in n for n in names), names
    assert rel_l2(dev_to_nchw(dx), oracle.conv_bwd_data(dy, w, (N, C, 1, 1), pad=0, stride=1)) <= TOL["f32"]
