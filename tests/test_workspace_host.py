"""Every convolution call takes the workspace that the query reports for it,
with and without a bias (CPU only).

Where no GPU can be reached, a call whose arguments pass every check ends at
its first launch with SINGA_ERR_HIP and touches nothing, so the checks alone
can be swept over many shapes with stand-in pointers.
"""
import ctypes
import itertools
import os

import pytest
import torch

from paper_1603_07846_amd import singa

pytestmark = pytest.mark.skipif(os.path.exists("/dev/kfd") or torch.cuda.device_count() > 0,
                                reason="stand-in pointers must not reach a GPU")

OK, WORKSPACE, HIP = 0, -4, -6
P = 1 << 20  # an aligned stand-in address

# (N, H, W, C, K, R, pad, stride): the extra column of a bias changes the tile
# count where R*R*C is a multiple of a tile's width
SHAPES = [s for s in itertools.product((1, 16, 50), (7, 14, 27), (7, 13), (3, 16, 30, 128, 512), (16, 96, 384), (1, 3, 5),
                                       (0, 1), (1, 2)) if s[5] <= min(s[1], s[2]) + 2 * s[6]]
SHAPES += [(50, 27, 27, 128, 16, 3, 1, 1), (64, 13, 13, 128, 16, 3, 1, 1), (32, 55, 55, 128, 16, 3, 1, 1),
           (16, 7, 7, 128, 96, 3, 1, 1), (16, 14, 14, 512, 384, 3, 1, 1), (2048, 1, 1, 14080, 1024, 1, 0, 1),
           (512, 1, 1, 14080, 1024, 1, 0, 1), (1, 1, 1, 4096, 4096, 1, 0, 1), (8, 57, 57, 3, 96, 11, 0, 4)]


class Call:
    """One geometry's call arguments; status(op, bias, ws_bytes) makes the call."""

    def __init__(self, dt, lay, shape):
        N, H, W, C, K, R, pad, stride = shape
        self.dt, self.lay = dt, lay
        self.xs = (N, C, H, W) if lay == singa.NCHW else (N, H, W, C)
        self.ws = (K, C, R, R) if lay == singa.NCHW else (K, R, R, C)
        self.geo = pad, stride
        self.x, self.w, self.d = (ctypes.byref(v) for v in (singa._act_shape4(self.xs, lay),
                                                            singa._filt4(self.ws, lay), singa._cdesc(pad, stride)))

    def reported(self, op):
        return singa.conv_workspace_bytes(op, self.dt, self.xs, self.ws, *self.geo, self.lay)

    def status(self, op, bias, nbytes):
        lib, b = singa.lib(), P if bias else None
        a, end = (self.dt, self.lay, self.x), (P if nbytes else None, nbytes, None)
        if op == singa.OP_FWD:
            return lib.singa_conv_fwd(*a, P, self.w, P, b, self.d, P, 0, *end)
        if op == singa.OP_BWD_DATA:
            return lib.singa_conv_bwd_data(*a, self.w, P, self.d, P, b, P, *end)
        if op == singa.OP_BWD_FILTER:
            return lib.singa_conv_bwd_filter(*a, P, self.w, self.d, P, P, b, 0, *end)
        return lib.singa_conv_bwd_filter_sgd(*a, P, self.w, self.d, P, None, None, P, P, None, b, b, None, 0.01, 0.9,
                                             0.0, *end)


OPS = {"fwd": singa.OP_FWD, "bwd_data": singa.OP_BWD_DATA, "bwd_filter": singa.OP_BWD_FILTER,
       "bwd_filter_sgd": singa.OP_BWD_FILTER_SGD}


@pytest.mark.parametrize("lay", [singa.NHWC, singa.NCHW], ids=["nhwc", "nchw"])
@pytest.mark.parametrize("dt", [singa.F32, singa.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("op", OPS)
def test_the_reported_workspace_is_enough(op, dt, lay):
    refused = []
    for shape in SHAPES:
        call = Call(dt, lay, shape)
        for bias in (True, False):
            rc = call.status(OPS[op], bias, call.reported(OPS[op]))
            assert rc in (HIP, WORKSPACE), (shape, bias, rc)
            if rc == WORKSPACE:
                refused.append((shape, bias))
    assert not refused, (len(refused), refused[:5])
