"""Convolution layers of any shape: the kernels for ragged images and channel
counts at the edges of their tiles (8 x 8 pixels and 64 channels forward, 8 x 16
pixels and 32 / 64 channels in the weight gradient), at rows of less than 8
pixels (loaded element by element), at every LDS size and beyond the largest,
with the checks and tolerances of the regular shapes, and at odd addresses against
even ones, bit for bit."""
import math

import pytest
import torch

import test_gpu_nn as T
from test_gpu_nn import nn  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

CASES = [
    (1, 2, 1, 1, 1),        # one pixel
    (2, 3, 2, 7, 7),        # rows below 8 pixels, channels below 4
    (1, 16, 64, 8, 8),      # one tile each way
    (2, 17, 65, 9, 8),      # one more of everything
    (1, 31, 33, 8, 17),
    (3, 64, 32, 15, 16),
    (1, 65, 63, 23, 9),
    (1, 129, 20, 10, 25),
    (1, 257, 9, 9, 33),
    (1, 384, 70, 14, 14),
    (1, 385, 10, 9, 15),    # beyond the staged halo
]


@pytest.mark.parametrize("n,cin,cout,h,w", CASES)
def test_forward(nn, n, cin, cout, h, w):  # noqa: F811
    T.test_conv_forward(nn, n, cin, cout, h, w)


@pytest.mark.parametrize("n,cin,cout,h,w", CASES)
def test_backward(nn, n, cin, cout, h, w):  # noqa: F811
    T.test_conv_backward(nn, n, cin, cout, h, w)
    T.test_conv_backward(nn, n, cout, cin, h, w)


@pytest.mark.parametrize("n,cin,cout,h,w", [(2, 20, 36, 13, 19), (1, 32, 64, 16, 16)])
def test_odd_addresses(nn, n, cin, cout, h, w):  # noqa: F811
    """x, the weights and dz one element past an even address: the ragged shape gives
    the same bits (its kernels do not depend on the alignment beyond the width of
    their loads); the regular shape's weight gradient is summed in the order of
    the same tiles and splits, so it does too."""
    g = torch.Generator().manual_seed(5)
    x = T.bits(torch.randn(cin, n, h, w, generator=g)).reshape(-1)
    dz = T.bits(torch.randn(cout, n, h, w, generator=g)).reshape(-1)
    wt = T.bits(torch.randn(cout, 9 * cin, generator=g) / math.sqrt(9 * cin)).reshape(-1)

    def odd(t):
        b = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
        b[1:1 + t.numel()] = t
        return b[1:1 + t.numel()]

    out = []
    for f in (lambda t: t, odd):
        xs, ws, ds = f(x), f(wt), f(dz)
        z = torch.empty(cout * n * h * w, device="cuda")
        dw, db = torch.empty(cout * cin * 9, device="cuda"), torch.empty(cout, device="cuda")
        work = torch.empty(nn.wgrad_work(n, cin, cout, h, w), device="cuda")
        if h % 16:  # (the regular forward's other order is within its own tolerance only)
            nn.conv3x3(xs, ws, None, n, cin, cout, h, w, z=z)
        else:
            z.zero_()
        nn.conv3x3_wgrad(xs, ds, dw, db, work, n, cin, cout, h, w)
        torch.cuda.synchronize()
        out.append((z.cpu(), dw.cpu()))
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("planes,h,w", [(1, 2, 2), (3, 6, 10), (5, 16, 24), (64, 32, 32)])
def test_pool_backward_join(nn, planes, h, w):  # noqa: F811
    """The joined gradient of a pooled and skipped activation against the three
    calls it replaces, bit for bit (the element-wise and the 16-byte kernels)."""
    g = torch.Generator().manual_seed(h + w)
    dy = torch.randn(planes * h * w // 4, generator=g).cuda()
    skip = torch.randn(planes * h * w, generator=g).cuda()
    a = T.bits(torch.relu(torch.randn(planes * h * w, generator=g)))
    dx, want = torch.empty_like(skip), torch.empty_like(a)
    nn.pool2_backward(dy, dx, planes, h, w)
    nn.axpy(1.0, skip, dx)
    nn.relu_bf16_backward(a, dx, want)
    got = torch.full_like(a, 0x7fff)
    nn.pool2_backward_join(dy, skip, a, got, planes, h, w)
    torch.cuda.synchronize()
    assert torch.equal(got.cpu(), want.cpu())
