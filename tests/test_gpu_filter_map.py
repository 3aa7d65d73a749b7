"""The filter gradient of layers whose GEMM result is laid out or shaped
otherwise than the caller's filter, with the reduction split (its writes go
through the map) and in one piece (staged): channel padding, space-to-depth,
KCRS filters and their combinations, written and accumulated."""
import pytest
import torch

import oracle
from _helpers import TOL, filt_to_kcrs, fphys, nchw_to_dev, rel_l2
from paper_1603_07846_amd import singa
from paper_1603_07846_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [  # (N, C, H, W, K, R, S, pad, stride)
    (8, 3, 24, 20, 16, 5, 5, 2, 1),     # colour channels padded to 4
    (9, 5, 17, 19, 24, 3, 3, 1, 1),     # 5 channels padded to 8
    (8, 3, 67, 61, 24, 11, 11, 0, 4),   # space-to-depth, taps past the filter's edge dropped
    (6, 3, 64, 50, 8, 7, 7, 3, 2),      # stride 2: space-to-depth in fp32, padded channels in bf16
    (8, 16, 23, 21, 40, 3, 5, 1, 1),    # no rewrite, non-square filter
    (32, 8, 16, 16, 264, 3, 3, 1, 2),   # strided, several row tiles
    (1, 3, 9, 9, 8, 3, 3, 1, 1),        # one piece: the staged path
    (1, 16, 6, 5, 12, 3, 3, 1, 1),
]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("layout", ["NHWC", "NCHW"])
@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_filter_gradient_reaches_the_callers_filter(case, layout, dt):
    N, C, H, W, K, R, S, pad, stride = case
    x = wl.random_array((N, C, H, W), 400, "normal", 1.0, dt)
    P, Q = oracle.conv_out(H, R, pad, stride), oracle.conv_out(W, S, pad, stride)
    dy = wl.random_array((N, K, P, Q), 401, "normal", 1.0, dt)
    ref_dw, ref_db = oracle.conv_bwd_filter(x, dy, (K, C, R, S), pad=pad, stride=stride)
    xd, dyd = nchw_to_dev(x, dt, layout), nchw_to_dev(dy, dt, layout)
    shape = fphys((K, C, R, S), layout)
    singa.trace_enable(True)
    dw, db = singa.conv_bwd_filter(xd, dyd, shape, pad, stride, layout=layout)
    torch.cuda.synchronize()
    names = [r[0] for r in singa.trace_records()]
    singa.trace_enable(False)
    moved = {"unpad_channels_f32_kernel", "s2d_to_filter_f32_kernel", "krsc_to_kcrs_kernel"} & set(names)
    rewritten = layout == "NCHW" or C % 4 != 0
    assert bool(moved) == (rewritten and "splitk_reduce_kernel" not in names), names
    assert rel_l2(filt_to_kcrs(dw, layout), ref_dw) <= TOL["f32"]
    assert rel_l2(db.cpu().numpy(), ref_db) <= TOL["f32"]
    singa.conv_bwd_filter(xd, dyd, shape, pad, stride, layout=layout, dw=dw, db=db, accumulate=True)
    torch.cuda.synchronize()
    assert rel_l2(filt_to_kcrs(dw, layout), 2 * ref_dw) <= TOL["f32"]
    assert rel_l2(db.cpu().numpy(), 2 * ref_db) <= TOL["f32"]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows", [(2, 5, 7), (1, 4, 2), (3, 8, 8)], ids=str)
def test_padded_input_and_filter_in_one_launch(rows, dt):
    """Colour channels padded to 4 for input and filter together, at pixel
    counts around the eight rows a thread moves."""
    N, H, W = rows
    case = (N, 3, H, W, 5, 1, 1, 0, 1)
    x = wl.random_array((N, 3, H, W), 410, "normal", 1.0, dt)
    w = wl.random_array((5, 3, 1, 1), 411, "normal", 1.0, dt)
    singa.trace_enable(True)
    y = singa.conv_fwd(nchw_to_dev(x, dt), torch.from_numpy(w.transpose(0, 2, 3, 1).copy()).cuda().to(
        torch.bfloat16 if dt == "bf16" else torch.float32), None, 0, 1)
    torch.cuda.synchronize()
    names = [r[0] for r in singa.trace_records()]
    singa.trace_enable(False)
    assert names.count("pad_channels_kernel") == 1, names
    ref = oracle.conv_fwd(x, w, None, pad=0, stride=1)
    assert rel_l2(y.float().cpu().numpy().transpose(0, 3, 1, 2), ref) <= TOL[dt], case
