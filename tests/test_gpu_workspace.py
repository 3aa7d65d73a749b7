"""Calls given exactly the workspace that the query reports, or that the
binding allocates by it, where a form without a bias takes more splits than
the one with it."""
import numpy as np
import pytest
import torch

import oracle
from paper_1603_07846_amd import singa
from paper_1603_07846_amd import workloads as wl
from _helpers import TOL, dev_to_nchw, filt_to_kcrs, gpu_full, kcrs_to_dev, nchw_to_dev, rel_l2, to_gpu
from test_workspace_host import OPS, least

pytestmark = pytest.mark.gpu

NO_BIAS = [("f32", (64, 128, 14, 14, 8, 1, 1, 1, 1)), ("f32", (512, 512, 4, 4, 8, 3, 3, 1, 1)),
           ("f32", (16, 128, 7, 7, 96, 3, 3, 1, 1)), ("bf16", (64, 256, 14, 14, 8, 3, 3, 1, 1))]


def _update(xd, dyd, wshape, dw, dt, pad, stride):
    """The fused call without a bias against the gradient dw and the flat update."""
    w0 = to_gpu(wl.random_array(wshape, 403, "normal", 0.1, "f32"))
    v0 = to_gpu(wl.random_array(wshape, 404, "normal", 0.01, "f32"))
    wr, vr, wf, vf = (to_gpu(t) for t in (w0, v0, w0, v0))
    wb = gpu_full(wshape, 0.0, torch.bfloat16)
    singa.sgd_momentum_update(wr, dw, vr, wb, 0.01, 0.9, 5e-4)
    wbf = gpu_full(wshape, 0.0, torch.bfloat16)
    singa.conv_bwd_filter_sgd(xd, dyd, wshape, wf, vf, wbf, lr=0.01, momentum=0.9, weight_decay=5e-4, pad=pad,
                              stride=stride)
    torch.cuda.synchronize()
    assert torch.equal(wf, wr) and torch.equal(vf, vr) and torch.equal(wbf, wb)


@pytest.mark.parametrize("dt,case", NO_BIAS, ids=[d + "-" + "x".join(map(str, c)) for d, c in NO_BIAS])
def test_gradient_and_update_without_a_bias(dt, case):
    N, C, H, W, K, R, S, pad, stride = case
    x = wl.random_array((N, C, H, W), 400, "normal", 1.0, dt)
    dy = wl.random_array((N, K, oracle.conv_out(H, R, pad, stride), oracle.conv_out(W, S, pad, stride)), 401, "normal",
                         1.0, dt)
    xd, dyd = nchw_to_dev(x, dt), nchw_to_dev(dy, dt)
    dw, _ = singa.conv_bwd_filter(xd, dyd, (K, R, S, C), pad, stride, with_bias=False)
    ref, _ = oracle.conv_bwd_filter(x, dy, (K, C, R, S), pad=pad, stride=stride)
    assert rel_l2(filt_to_kcrs(dw), ref) <= TOL[dt]
    _update(xd, dyd, (K, R, S, C), dw, dt, pad, stride)


def test_update_fused_with_and_without_a_bias():
    """A dense layer of 440 gradient tiles: with a bias column they are 448,
    one split, and the update is fused; without it the same."""
    N, C, K = 512, 14080, 1024
    assert singa.conv_workspace_bytes(singa.OP_BWD_FILTER_SGD, singa.BF16, (N, 1, 1, C), (K, 1, 1, C)) == 0
    x = wl.random_array((N, 1, 1, C), 405, "normal", 1.0, "bf16")
    dy = wl.random_array((N, 1, 1, K), 406, "normal", 1.0, "bf16")
    xd, dyd = to_gpu(x, torch.bfloat16), to_gpu(dy, torch.bfloat16)
    dw, _ = singa.conv_bwd_filter(xd, dyd, (K, 1, 1, C), with_bias=False)
    ref = dy.reshape(N, K).astype(np.float64).T @ x.reshape(N, C).astype(np.float64)
    assert rel_l2(dw.cpu().numpy().reshape(K, C), ref) <= TOL["f32"]  # fp32 sums of bf16 products
    _update(xd, dyd, (K, 1, 1, C), dw, "bf16", 0, 1)


def test_fixed_array_makes_the_splits_of_the_workspace_call():
    """An fp32 gradient whose time model would like 138 MB of partial sums:
    limited to the fixed array's size for both calls, and the same bits."""
    N, C, H, K = 128, 1024, 13, 1024
    assert singa.conv_workspace_bytes(singa.OP_BWD_FILTER, singa.F32, (N, H, H, C), (K, 1, 1, C)) \
        <= singa.NOALLOC_SCRATCH_BYTES
    xd = to_gpu(wl.random_array((N, H, H, C), 410, "normal", 1.0, "f32"))
    dyd = to_gpu(wl.random_array((N, H, H, K), 411, "normal", 1.0, "f32"))
    dw, db = singa.conv_bwd_filter(xd, dyd, (K, 1, 1, C))
    dn, bn = singa.conv_bwd_filter_noalloc(xd, dyd, (K, 1, 1, C))
    torch.cuda.synchronize()
    assert torch.equal(dw, dn) and torch.equal(db, bn)


LEAST = [("fwd", (1, 128, 14, 7, 16, 3, 3, 1, 1)), ("bwd_data", (1, 16, 27, 13, 16, 5, 5, 0, 1)),
         ("bwd_filter", (50, 16, 14, 13, 16, 1, 1, 1, 1)), ("bwd_filter", (1, 128, 14, 13, 96, 1, 1, 1, 1)),
         ("bwd_filter_sgd", (50, 16, 14, 13, 16, 1, 1, 1, 1))]


@pytest.mark.parametrize("op,case", LEAST, ids=[o + "-" + "x".join(map(str, c)) for o, c in LEAST])
def test_f32_calls_with_the_least_workspace(op, case):
    """Fewer splits than with the reported size; the workspace's guard bands
    stay whole, and one byte less is refused."""
    N, C, H, W, K, R, S, pad, stride = case
    code = OPS[op]
    need = least(code, (N, H, W, C, K, R, pad, stride), True)
    assert need < singa.conv_workspace_bytes(code, singa.F32, (N, H, W, C), (K, R, S, C), pad, stride)
    x = wl.random_array((N, C, H, W), 420, "normal", 1.0, "f32")
    w = wl.random_array((K, C, R, S), 421, "normal", 0.05, "f32")
    dy = wl.random_array((N, K, oracle.conv_out(H, R, pad, 1), oracle.conv_out(W, S, pad, 1)), 422, "normal", 1.0, "f32")
    b = wl.random_array((K,), 423, "normal", 0.1, "f32")
    xd, wd, dyd, bd = nchw_to_dev(x), kcrs_to_dev(w), nchw_to_dev(dy), to_gpu(b)
    ref_dw, ref_db = oracle.conv_bwd_filter(x, dy, w.shape, pad=pad, stride=1)

    def run(nbytes):
        ws = singa.empty((max(nbytes, 1),), torch.uint8, "cuda")[:nbytes]
        if op == "fwd":
            return dev_to_nchw(singa.conv_fwd(xd, wd, bd, pad, 1, workspace=ws)), oracle.conv_fwd(x, w, b, pad=pad,
                                                                                                stride=1)
        if op == "bwd_data":
            return dev_to_nchw(singa.conv_bwd_data(dyd, wd, xd.shape, pad, 1, workspace=ws)), oracle.conv_bwd_data(
                dy, w, x.shape, pad=pad, stride=1)
        dw, db = gpu_full((K, R, S, C), 0.0), gpu_full((K,), 0.0)
        if op == "bwd_filter":
            singa.conv_bwd_filter(xd, dyd, dw.shape, pad, 1, dw=dw, db=db, workspace=ws)
            return filt_to_kcrs(dw), ref_dw
        wf, vf, bf, vbf = (to_gpu(t) for t in (wd, wd, bd, bd))
        singa.conv_bwd_filter_sgd(xd, dyd, dw.shape, wf, vf, b=bf, vb=vbf, lr=0.01, momentum=0.9, pad=pad, dw=dw, db=db,
                                  workspace=ws)
        ref_w, _ = oracle.sgd_momentum(w, ref_dw, w, 0.01, 0.9, 0.0)
        assert rel_l2(filt_to_kcrs(wf), ref_w) <= TOL["f32"] and rel_l2(db.cpu().numpy(), ref_db) <= TOL["f32"]
        return filt_to_kcrs(dw), ref_dw

    got, ref = run(need)
    torch.cuda.synchronize()
    assert rel_l2(got, ref) <= TOL["f32"]
    if need > 0:
        with pytest.raises(singa.SingaError) as e:
            run(need - 1)
        assert e.value.status == -4
