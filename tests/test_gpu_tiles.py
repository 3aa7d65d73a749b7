"""Every tile of the direct-to-LDS forward kernel against the oracle.

Each case is small but takes one tile (checked through the kernel trace) in
one way of summing the taps: in one piece ("one"), in several pieces that a
workgroup adds in order ("seg", bf16), or in one piece per workgroup with a
reduction after it ("split").  Rows, columns and taps are ragged; channel
counts are multiples of a K-tile, of a vector only, or in between.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1603_07846_amd import singa
from paper_1603_07846_amd import workloads as wl
from _helpers import TOL, dev_to_nchw, kcrs_to_dev, nchw_to_dev, phys, rel_l2

pytestmark = pytest.mark.gpu

CASES = [  # dtype, tile, summation, (N, C, H, W, K, R, S, pad, stride)
    ("bf16", "128x128", "one", (48, 16, 30, 25, 77, 1, 1, 0, 1)),
    ("bf16", "128x128", "split", (8, 168, 18, 20, 137, 5, 5, 2, 1)),
    ("bf16", "128x32", "one", (16, 16, 26, 26, 93, 1, 1, 0, 1)),
    ("bf16", "128x32", "seg", (48, 56, 4, 23, 198, 3, 3, 1, 1)),
    ("bf16", "128x32", "split", (3, 352, 35, 10, 8, 5, 5, 2, 1)),
    ("bf16", "128x64", "one", (31, 8, 30, 21, 161, 1, 1, 0, 1)),
    ("bf16", "128x64", "split", (48, 208, 7, 17, 33, 3, 3, 1, 1)),
    ("bf16", "192x128", "one", (64, 32, 40, 14, 76, 5, 5, 2, 1)),
    ("bf16", "192x128", "split", (2, 216, 30, 37, 68, 5, 5, 2, 1)),
    ("bf16", "256x128", "one", (64, 24, 15, 27, 148, 5, 5, 2, 1)),
    ("bf16", "256x128", "split", (31, 280, 28, 3, 135, 3, 3, 1, 1)),
    ("bf16", "256x64", "one", (64, 8, 31, 37, 44, 1, 1, 0, 1)),
    ("bf16", "256x64", "split", (64, 328, 4, 27, 36, 3, 3, 1, 1)),
    ("bf16", "32x128", "seg", (2, 200, 34, 40, 384, 3, 3, 1, 1)),
    ("bf16", "32x128", "split", (2, 144, 21, 16, 106, 5, 5, 2, 1)),
    ("bf16", "64x128", "one", (31, 8, 37, 26, 97, 1, 1, 0, 1)),
    ("bf16", "64x128", "seg", (24, 64, 25, 20, 168, 3, 3, 1, 1)),
    ("bf16", "64x128", "split", (12, 80, 9, 13, 163, 5, 5, 2, 1)),
    ("bf16", "64x64", "one", (2, 8, 7, 4, 57, 1, 1, 0, 1)),
    ("bf16", "64x64", "seg", (3, 56, 6, 4, 13, 3, 3, 1, 1)),
    ("bf16", "64x64", "split", (1, 80, 10, 12, 19, 3, 3, 1, 1)),
    ("f32", "128x128", "one", (8, 4, 25, 30, 355, 1, 1, 0, 1)),
    ("f32", "128x128", "split", (12, 180, 36, 39, 106, 3, 3, 1, 1)),
    ("f32", "128x32", "one", (24, 36, 36, 21, 9, 1, 1, 0, 1)),
    ("f32", "128x32", "split", (5, 144, 39, 12, 8, 3, 3, 1, 1)),
    ("f32", "128x64", "one", (24, 4, 31, 28, 35, 3, 3, 1, 1)),
    ("f32", "128x64", "split", (3, 152, 36, 26, 38, 3, 3, 1, 1)),
    ("f32", "192x128", "one", (48, 28, 40, 8, 309, 3, 3, 1, 1)),
    ("f32", "192x128", "split", (24, 36, 36, 13, 78, 5, 5, 2, 1)),
    ("f32", "256x128", "one", (48, 32, 34, 12, 366, 3, 3, 1, 1)),
    ("f32", "256x128", "split", (64, 80, 15, 19, 101, 3, 3, 1, 1)),
    ("f32", "256x64", "one", (31, 8, 32, 36, 48, 1, 1, 0, 1)),
    ("f32", "256x64", "split", (12, 80, 38, 31, 142, 3, 3, 1, 1)),
    ("f32", "32x128", "one", (3, 156, 25, 36, 356, 1, 1, 0, 1)),
    ("f32", "32x128", "split", (2, 184, 5, 27, 199, 3, 3, 1, 1)),
    ("f32", "64x128", "one", (8, 4, 34, 29, 158, 1, 1, 0, 1)),
    ("f32", "64x128", "split", (12, 120, 5, 22, 66, 5, 5, 2, 1)),
    ("f32", "64x64", "one", (3, 8, 7, 4, 40, 1, 1, 0, 1)),
    ("f32", "64x64", "split", (1, 176, 6, 12, 21, 1, 1, 0, 1)),
]


def _data(case, dt, seed):
    N, C, H, W, K, R, S, pad, stride = case
    x = wl.random_array((N, C, H, W), seed, "normal", 1.0, dt)
    w = wl.random_array((K, C, R, S), seed + 1, "normal", 0.1, dt)
    b = wl.random_array((K,), seed + 2, "normal", 0.5, "f32")
    return x, w, b


@pytest.mark.parametrize("dt,tile,how,case", CASES,
                         ids=["-".join(c[:3]) + "-" + "x".join(map(str, c[3])) for c in CASES])
def test_forward_tile(dt, tile, how, case):
    N, C, H, W, K, R, S, pad, stride = case
    x, w, b = _data(case, dt, 300)
    singa.trace_enable(True)
    y = singa.conv_fwd(nchw_to_dev(x, dt), kcrs_to_dev(w, dt), torch.from_numpy(b).cuda(), pad, stride, relu=True)
    torch.cuda.synchronize()
    names = [r[0] for r in singa.trace_records()]
    singa.trace_enable(False)
    assert "conv_fwd_kernel<%s,%s,0>" % (dt, tile) in names, names
    assert ("splitk_epilogue_kernel" in names) == (how == "split"), names
    ref = oracle.relu_fwd(oracle.conv_fwd(x, w, b, pad=pad, stride=stride))
    assert rel_l2(dev_to_nchw(y), ref) <= TOL[dt]


# the source gradient: the same kernel with a folded ReLU mask, at stride 1
# and 2 (the latter on the space-to-depth layer)
BWD_CASES = [(3, 40, 14, 11, 72, 3, 3, 1, 1), (2, 64, 13, 13, 128, 5, 5, 2, 1), (6, 96, 9, 9, 200, 1, 1, 0, 1),
             (3, 24, 15, 13, 64, 3, 3, 1, 2)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", BWD_CASES, ids=["x".join(map(str, c)) for c in BWD_CASES])
def test_source_gradient_tile(case, dt):
    N, C, H, W, K, R, S, pad, stride = case
    x, w, _ = _data(case, dt, 310)
    xr = np.maximum(x, 0.0)
    P, Q = oracle.conv_out(H, R, pad, stride), oracle.conv_out(W, S, pad, stride)
    dy = wl.random_array((N, K, P, Q), 313, "normal", 1.0, dt)
    singa.trace_enable(True)
    dx = singa.conv_bwd_data(nchw_to_dev(dy, dt), kcrs_to_dev(w, dt), phys(x.shape), pad, stride,
                             relu_y=nchw_to_dev(xr, dt))
    torch.cuda.synchronize()
    names = [r[0] for r in singa.trace_records()]
    singa.trace_enable(False)
    assert any(n.startswith("conv_fwd_kernel<%s," % dt) and "x" in n.split(",")[1] for n in names), names
    ref = oracle.relu_bwd(xr, oracle.conv_bwd_data(dy, w, x.shape, pad=pad, stride=stride))
    got = dev_to_nchw(dx)
    np.testing.assert_array_equal(got[xr <= 0], 0.0)
    assert rel_l2(got, ref) <= TOL[dt]


# the fp32 filter gradient's tiles: rows of the tile, how the reduction is
# summed, whether a K-tile is 32 images at one pixel, and the layer (strided
# and channel-padded ones among them)
WGRAD_CASES = [
    (32, "one", 0, (1, 44, 3, 15, 28, 3, 3, 1, 1)),
    (32, "one", 1, (32, 148, 7, 1, 20, 1, 1, 0, 1)),
    (32, "split", 0, (8, 4, 7, 20, 92, 1, 1, 0, 1)),
    (32, "split", 1, (64, 28, 14, 5, 4, 1, 1, 0, 1)),
    (64, "one", 0, (1, 116, 5, 1, 404, 5, 5, 2, 1)),
    (64, "one", 1, (32, 156, 2, 1, 280, 5, 5, 2, 1)),
    (64, "split", 0, (31, 4, 6, 12, 392, 1, 1, 0, 1)),
    (64, "split", 1, (32, 4, 4, 18, 344, 1, 1, 0, 1)),
    (128, "one", 0, (5, 156, 1, 24, 520, 5, 5, 2, 1)),
    (128, "split", 0, (12, 4, 22, 20, 444, 1, 1, 0, 1)),
    (128, "split", 1, (32, 4, 15, 24, 184, 1, 1, 0, 1)),
    (32, "split", 0, (3, 3, 32, 32, 32, 5, 5, 2, 1)),    # 3 channels padded to 4
    (32, "split", 0, (5, 32, 15, 17, 24, 3, 3, 1, 2)),   # stride 2
]


@pytest.mark.parametrize("bias", [True, False], ids=["bias", "no-bias"])
@pytest.mark.parametrize("rows,how,nfast,case", WGRAD_CASES,
                         ids=["%d-%s-%d-" % c[:3] + "x".join(map(str, c[3])) for c in WGRAD_CASES])
def test_f32_filter_gradient_tile(rows, how, nfast, case, bias):
    N, C, H, W, K, R, S, pad, stride = case
    x, w, _ = _data(case, "f32", 320)
    P, Q = oracle.conv_out(H, R, pad, stride), oracle.conv_out(W, S, pad, stride)
    dy = wl.random_array((N, K, P, Q), 323, "normal", 1.0, "f32")
    xd, dyd = nchw_to_dev(x, "f32"), nchw_to_dev(dy, "f32")
    ref_dw, ref_db = oracle.conv_bwd_filter(x, dy, w.shape, pad=pad, stride=stride)
    wshape = (K, R, S, C)
    singa.trace_enable(True)
    dw, db = singa.conv_bwd_filter(xd, dyd, wshape, pad, stride, with_bias=bias)
    torch.cuda.synchronize()
    names = [r[0] for r in singa.trace_records()]
    singa.trace_enable(False)
    assert "conv_wgrad_kernel<f32,%dx128,%d>" % (rows, nfast) in names, names
    assert ("splitk_reduce_kernel" in names) == (how == "split"), names
    assert rel_l2(dw.cpu().numpy().transpose(0, 3, 1, 2), ref_dw) <= TOL["f32"]
    # accumulated: once more on top, and through the fixed scratch array
    singa.conv_bwd_filter(xd, dyd, wshape, pad, stride, dw=dw, db=db, accumulate=True, with_bias=bias)
    dn, bn = singa.conv_bwd_filter_noalloc(xd, dyd, wshape, pad, stride, with_bias=bias)
    torch.cuda.synchronize()
    assert rel_l2(dw.cpu().numpy().transpose(0, 3, 1, 2), 2 * ref_dw) <= TOL["f32"]
    assert rel_l2(dn.cpu().numpy().transpose(0, 3, 1, 2), ref_dw) <= TOL["f32"]
    if bias:
        assert rel_l2(db.cpu().numpy(), 2 * ref_db) <= TOL["f32"]
        assert rel_l2(bn.cpu().numpy(), ref_db) <= TOL["f32"]


def test_f32_filter_gradient_least_workspace():
    """A workspace of the size that the least number of partial tiles takes
    (what the register-staged kernel's split rule asks for) is still enough."""
    N, C, H, W, K, R, S, pad, stride = case = (2, 96, 19, 19, 144, 5, 5, 0, 1)  # 450 pixels: that rule has one split
    x, w, _ = _data(case, "f32", 330)
    dy = wl.random_array((N, K, 15, 15), 333, "normal", 1.0, "f32")
    xd, dyd = nchw_to_dev(x, "f32"), nchw_to_dev(dy, "f32")
    assert singa.conv_workspace_bytes(singa.OP_BWD_FILTER, torch.float32, phys(x.shape), (K, R, S, C), pad, stride) > 0
    ref_dw, ref_db = oracle.conv_bwd_filter(x, dy, w.shape, pad=pad, stride=stride)
    ws = torch.empty(16, dtype=torch.uint8, device="cuda")
    dw, db = singa.conv_bwd_filter(xd, dyd, (K, R, S, C), pad, stride, workspace=ws)
    torch.cuda.synchronize()
    assert rel_l2(dw.cpu().numpy().transpose(0, 3, 1, 2), ref_dw) <= TOL["f32"]
    assert rel_l2(db.cpu().numpy(), ref_db) <= TOL["f32"]


# the bf16 filter gradient of few filters: one or two of a tile's four
# 32-filter blocks in use, at their edges and one past; summed in one piece
# and split, K-tiles of 32 images at one pixel (N = 32) and across pixels
NARROW_CASES = [(32, 16, 6, 5, 8, 3, 3, 1, 1), (3, 40, 9, 7, 32, 1, 1, 0, 1), (5, 24, 11, 8, 40, 5, 5, 2, 1),
                (32, 72, 4, 4, 64, 3, 3, 1, 1), (7, 8, 13, 13, 64, 3, 3, 0, 2), (1, 32, 3, 3, 24, 1, 1, 0, 1),
                (1, 264, 4, 4, 56, 1, 1, 0, 1), (32, 16, 6, 5, 72, 3, 3, 1, 1)]


@pytest.mark.parametrize("bias", [True, False], ids=["bias", "no-bias"])
@pytest.mark.parametrize("case", NARROW_CASES, ids=["x".join(map(str, c)) for c in NARROW_CASES])
def test_bf16_filter_gradient_of_few_filters(case, bias):
    N, C, H, W, K, R, S, pad, stride = case
    x, w, _ = _data(case, "bf16", 340)
    P, Q = oracle.conv_out(H, R, pad, stride), oracle.conv_out(W, S, pad, stride)
    dy = wl.random_array((N, K, P, Q), 343, "normal", 1.0, "bf16")
    ref_dw, ref_db = oracle.conv_bwd_filter(x, dy, w.shape, pad=pad, stride=stride)
    singa.trace_enable(True)
    dw, db = singa.conv_bwd_filter(nchw_to_dev(x, "bf16"), nchw_to_dev(dy, "bf16"), (K, R, S, C), pad, stride,
                                   with_bias=bias)
    torch.cuda.synchronize()
    names = [r[0] for r in singa.trace_records()]
    singa.trace_enable(False)
    assert any(n.startswith("conv_wgrad_large_kernel<") for n in names), names
    assert rel_l2(dw.cpu().numpy().transpose(0, 3, 1, 2), ref_dw) <= TOL["bf16"]
    if bias:
        assert rel_l2(db.cpu().numpy(), ref_db) <= TOL["bf16"]


# dense layers of one to three rows: the matrix-vector kernel, at widths
# around its four columns a workgroup and reductions around the 256 chunks
# that it takes at a time; four rows take a tile
GEMV_CASES = [(1, 16, 4, 4, 1), (2, 40, 1, 1, 7), (3, 8, 5, 3, 10), (1, 4096, 1, 1, 130), (2, 264, 4, 4, 33),
              (3, 2048, 1, 1, 1000), (4, 2048, 1, 1, 100)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("relu", [False, True], ids=["", "relu"])
@pytest.mark.parametrize("case", GEMV_CASES, ids=["x".join(map(str, c)) for c in GEMV_CASES])
def test_dense_layer_of_few_rows(case, relu, dt):
    N, C, H, W, K = case
    x, w, b = _data((N, C, H, W, K, H, W, 0, 1), dt, 340)
    singa.trace_enable(True)
    y = singa.conv_fwd(nchw_to_dev(x, dt), kcrs_to_dev(w, dt), torch.from_numpy(b).cuda() if relu else None, 0, 1,
                       relu=relu)
    torch.cuda.synchronize()
    names = [r[0] for r in singa.trace_records()]
    singa.trace_enable(False)
    assert (names == ["conv_fwd_kernel<%s,gemv,0>" % dt]) == (N <= 3), names
    ref = oracle.conv_fwd(x, w, b if relu else None, pad=0, stride=1)
    ref = oracle.relu_fwd(ref) if relu else ref
    assert rel_l2(dev_to_nchw(y), ref) <= TOL[dt]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_source_gradient_of_few_rows(dt):
    """fp32 backward-data runs the matrix-vector kernel on the transposed
    weights, with the ReLU below folded in."""
    N, C, H, W, K = 2, 24, 3, 3, 40
    x, w, _ = _data((N, C, H, W, K, H, W, 0, 1), dt, 350)
    xr = np.maximum(x, 0.0)
    dy = wl.random_array((N, K, 1, 1), 353, "normal", 1.0, dt)
    dx = singa.conv_bwd_data(nchw_to_dev(dy, dt), kcrs_to_dev(w, dt), phys(x.shape), 0, 1, relu_y=nchw_to_dev(xr, dt))
    torch.cuda.synchronize()
    ref = oracle.relu_bwd(xr, oracle.conv_bwd_data(dy, w, x.shape, pad=0, stride=1))
    got = dev_to_nchw(dx)
    np.testing.assert_array_equal(got[xr <= 0], 0.0)
    assert rel_l2(got, ref) <= TOL[dt]
