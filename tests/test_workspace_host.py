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


# ------------------------------------------------- what fp32 has to have
#
# The least that an fp32 call works with is what the split counts of the
# register-staged 128 x 128 kernels take, written down here once more.

def _up(v):
    return (v + 255) // 256 * 256


def _cd(a, b):
    return -(-a // b)


def _gemm_least(M, Nn, Kg):
    tiles, nkt = _cd(M, 128) * _cd(Nn, 128), _cd(Kg, 32)
    splits = 1 if tiles >= 256 or nkt < 8 else min(_cd(512, tiles), nkt // 4, 16)
    splits = _cd(nkt, _cd(nkt, splits)) if splits > 1 else 1
    return _up(4 * splits * M * Nn) if splits > 1 else 0


def _gradient_least(M, Ng, T):
    tiles, nkt = _cd(M, 128) * _cd(Ng, 128), _cd(T, 32)
    splits = min(max(min(_cd(1024, tiles), nkt // 8), 1), 256)
    splits = _cd(nkt, _cd(nkt, splits))
    return _up(4 * splits * M * _cd(Ng, 64) * 64) if splits > 1 else 0


def least(op, shape, bias):
    """Stride 1, NHWC, channels and filters in vectors of four."""
    N, H, W, C, K, R, pad, _ = shape
    Po, Qo, filt = H + 2 * pad - R + 1, W + 2 * pad - R + 1, 4 * K * R * R * C
    if op == singa.OP_FWD:
        return _gemm_least(N * Po * Qo, K, R * R * C)
    if op == singa.OP_BWD_DATA:
        dense = Po == Qo == 1 and pad == 0
        M, Nn, Kg = (N, R * R * C, K) if dense else (N * H * W, C, R * R * K)
        return _up(filt) + _gemm_least(M, Nn, Kg)
    g = _gradient_least(K, R * R * C + bias, N * Po * Qo)
    return g if op == singa.OP_BWD_FILTER else _up(filt) + (_up(4 * K) if bias else 0) + g


PLAIN = [s for s in SHAPES if s[7] == 1 and s[3] % 4 == 0 and s[4] % 4 == 0]
PLAIN += [(256, 24, 24, 1792, 320, 5, 2, 1), (128, 13, 13, 1024, 1024, 1, 0, 1), (32, 27, 27, 1024, 1024, 1, 0, 1),
          (2, 19, 19, 96, 144, 5, 0, 1), (250, 32, 32, 8, 32, 5, 2, 1)]


@pytest.mark.parametrize("op", OPS)
def test_f32_works_with_the_least_and_asks_for_little_more(op):
    more = 0
    for shape in PLAIN:
        call = Call(singa.F32, singa.NHWC, shape)
        need = [least(OPS[op], shape, bias) for bias in (False, True)]
        for bias in (False, True):
            assert call.status(OPS[op], bias, need[bias]) == HIP, (shape, bias)
            if need[bias] > 0:
                assert call.status(OPS[op], bias, need[bias] - 1) == WORKSPACE, (shape, bias)
        grown = call.reported(OPS[op]) - max(need)
        assert 0 <= grown <= 128 << 20, (shape, grown)
        more += grown > 0
    assert more > 0  # the range holds calls that ask for more


def test_f32_gradient_in_the_fixed_array():
    """The allocation-free call takes the whole of what the call with a
    workspace takes, or is refused where even the least does not fit."""
    lib = singa.lib()

    def noalloc(call, bias):
        return lib.singa_conv_bwd_filter_noalloc(call.dt, call.lay, call.x, P, call.w, call.d, P, P,
                                                 P if bias else None, 0, None)
    big = [(n, h, h, c, k, r, r // 2, 1) for n, h, c, k, r in
           itertools.product((8, 32, 64, 128), (13, 27), (128, 512, 1024), (64, 384, 1024), (1, 3, 5))]
    for shape in PLAIN + big:
        call = Call(singa.F32, singa.NHWC, shape)
        for bias in (False, True):
            assert least(singa.OP_BWD_FILTER, shape, bias) <= singa.NOALLOC_SCRATCH_BYTES
            assert noalloc(call, bias) == HIP, (shape, bias)
        assert call.reported(singa.OP_BWD_FILTER) <= singa.NOALLOC_SCRATCH_BYTES
    # permuted activations alone pass the array's size
    for bias in (False, True):
        assert noalloc(Call(singa.F32, singa.NCHW, (256, 55, 55, 64, 64, 3, 1, 1)), bias) == -7
