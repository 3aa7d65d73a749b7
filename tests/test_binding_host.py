"""The binding's declared arguments against the C header, its per-geometry
plans, and the calls on another stream that it refuses (CPU only)."""
import ctypes
import os
import re

import pytest
import torch

from paper_1603_07846_amd import singa

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "singa_mi.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    for m in re.finditer(r"\b(?:int|const char\*)\s+(singa_\w+)\(([^;]*)\);", text):
        args = [a.strip() for a in m.group(2).replace("\n", " ").split(",")]
        yield m.group(1), [] if args == ["void"] else args


@pytest.mark.parametrize("name,args", list(_declared()), ids=[n for n, _ in _declared()])
def test_argument_types_follow_the_header(name, args):
    """Every call declares every argument; a pointer (or stream) is never
    passed as an int, which would cut it to 32 bits."""
    types = getattr(singa.lib(), name).argtypes
    assert types is not None and len(types) == len(args)
    for arg, t in zip(args, types):
        pointer = "*" in arg or "singa_stream" in arg
        assert pointer == (t in (ctypes.c_void_p, ctypes.c_char_p) or hasattr(t, "_type_") and not
                           isinstance(t._type_, str)), (name, arg, t)
        if "float " in arg and not pointer:
            assert t is ctypes.c_float, (name, arg)
        if "size_t " in arg and not pointer:
            assert t is ctypes.c_size_t, (name, arg)


def test_plans_repeat_and_refuse():
    for _ in range(2):  # the second time from the kept plan
        assert singa.conv_out_shape((2, 9, 9, 8), (16, 3, 3, 8), 1, 2) == (2, 5, 5, 16)
        assert singa.conv_out_shape([2, 9, 9, 8], [16, 3, 3, 8], [1, 1], (2, 2)) == (2, 5, 5, 16)
        assert singa.conv_out_shape((2, 8, 9, 9), (16, 8, 3, 3), 1, 2, layout="NCHW") == (2, 16, 5, 5)
        assert singa.pool_out_shape((1, 13, 13, 4), "max") == (1, 6, 6, 4)
        with pytest.raises(singa.SingaError) as e:
            singa.conv_out_shape((2, 9, 9, 8), (16, 3, 3, 7))
        assert e.value.status == -2
        with pytest.raises(singa.SingaError) as e:
            singa.pool_out_shape((1, 13, 13, 4), "max", k=3, pad=3)
        assert e.value.status == -3


@pytest.mark.parametrize("missing", ["dw", "db", "workspace"])
def test_another_stream_needs_its_buffers(missing):
    """A buffer allocated by the call would belong to the current stream."""
    x, dy = torch.zeros(64, 9, 9, 16), torch.zeros(64, 9, 9, 24)
    kw = dict(dw=torch.zeros(24, 3, 3, 16), db=torch.zeros(24), workspace=torch.zeros(1 << 24, dtype=torch.uint8))
    assert singa.conv_workspace_bytes(singa.OP_BWD_FILTER, torch.float32, x.shape, (24, 3, 3, 16), 1) > 0
    kw[missing] = None
    with pytest.raises(ValueError):
        singa.conv_bwd_filter(x, dy, (24, 3, 3, 16), 1, on=object(), **kw)


def test_backward_that_raises_keeps_no_stream(monkeypatch):
    """The stream looked up for a backward pass is not the one of a later
    call when the pass ends in an exception."""
    from paper_1603_07846_amd import net as gnet

    class Broken:
        def compute_gradient(self, g, need_dx):
            raise RuntimeError("layer")

    net = object.__new__(gnet.Net)
    net.device, net.layers, net.side_update_layers = torch.device("cuda", 0), [Broken()], []
    net.wgrad_stream = object()
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: object())
    with pytest.raises(RuntimeError, match="layer"):
        net.backward()
    assert net.main_stream is None
