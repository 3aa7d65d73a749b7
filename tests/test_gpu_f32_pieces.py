"""fp32 sums over long ranges run in pieces of at most 256 terms whatever the
splits, so their rounding error does not grow with a split's length."""
import pytest
import torch

from paper_1603_07846_amd import singa

pytestmark = pytest.mark.gpu


def _bound(terms):
    """Each of a running sum's j-th additions of zero-mean terms rounds a value
    of size sqrt(j) by at most 2^-24 of it: relative to the final sqrt(n) that
    is 2^-24 sqrt(n / 2) in the 2-norm.  Pieces of 256, then their sums."""
    return 2.0 ** -24 * ((256 / 2) ** 0.5 + (terms / 256 / 2) ** 0.5 + 1)


def _rel(got, want):
    return float((got.double() - want).norm() / want.norm())


# rows, taps, filters: pieces exact, ragged and with one K-tile left over; the
# first fill the chip without a split
@pytest.mark.parametrize("n,c,k", [(8450, 2048, 512), (8450, 2084, 516), (4225, 4096, 384), (1000, 4136, 256)])
def test_forward_and_filter_gradient(n, c, k):
    g = torch.Generator(device="cuda").manual_seed(n + c)
    x = torch.randn((n, 1, 1, c), generator=g, device="cuda")
    w = torch.randn((k, 1, 1, c), generator=g, device="cuda")
    dy = torch.randn((n, 1, 1, k), generator=g, device="cuda")
    x64, w64, dy64 = (t.flatten(1).double() for t in (x, w, dy))
    y = singa.conv_fwd(x, w).flatten(1)
    dx = singa.conv_bwd_data(dy, w, x.shape).flatten(1)
    dw, db = singa.conv_bwd_filter(x, dy, tuple(w.shape))
    assert _rel(y, x64 @ w64.t()) <= _bound(c)
    assert _rel(dx, dy64 @ w64) <= _bound(k)
    assert _rel(dw.flatten(1), dy64.t() @ x64) <= _bound(n)
    assert _rel(db, dy64.sum(0)) <= _bound(n)


def test_pieces_of_a_convolution():
    """Image by image and image-fastest reductions of a 3x3 layer (N = 50 and
    64), through the whole-window taps."""
    for n in (50, 64):
        g = torch.Generator(device="cuda").manual_seed(n)
        x = torch.randn((n, 13, 13, 96), generator=g, device="cuda")
        dy = torch.randn((n, 11, 11, 100), generator=g, device="cuda")
        dw, _ = singa.conv_bwd_filter(x, dy, (100, 3, 3, 96), with_bias=False)
        d = dy.double().flatten(0, 2).t()
        want = torch.stack([d @ x[:, r:r + 11, s:s + 11].double().flatten(0, 2) for r in range(3) for s in range(3)], 1)
        assert _rel(dw.flatten(1), want.flatten(1)) <= _bound(n * 121)
