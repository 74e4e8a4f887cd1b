"""Convolutions whose inputs lie where the kernels' wide loads would not expect them."""
import math

import pytest
import torch

import test_gpu_nn as T
from test_gpu_nn import nn  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def shifted(t, by):
    b = torch.full((t.numel() + 8,), 0x7fc0, dtype=t.dtype, device="cuda")
    b[by:by + t.numel()] = t.reshape(-1)
    return b[by:by + t.numel()]


@pytest.mark.parametrize("n,cin,cout,h,w", [(2, 32, 64, 16, 16), (1, 32, 33, 48, 32), (3, 64, 70, 32, 16),
                                             (1, 416, 20, 16, 32)])
@pytest.mark.parametrize("by", [1, 4])
def test_regular_shape_with_x_off_a_16_byte_address(nn, n, cin, cout, h, w, by):  # noqa: F811
    """Forward and data gradient of a regular shape do not depend on where x lies: the
    same bits as at an aligned address (one chunk of channels, several, beyond 384)."""
    g = torch.Generator().manual_seed(cin)
    x = T.bits(T.bf16_round(torch.randn(cin, n, h, w, generator=g)))
    wt = T.bits(T.bf16_round(torch.randn(cout, 9 * cin, generator=g) / math.sqrt(9 * cin)))
    bias = torch.randn(cout, generator=g).cuda()
    act = T.bits(torch.relu(torch.randn(cout, n, h, w, generator=g)))
    out = []
    for xs in (x.reshape(-1), shifted(x, by)):
        z = torch.empty(cout * n * h * w, device="cuda")
        a = torch.empty(cout * n * h * w, dtype=torch.int16, device="cuda")
        dza = torch.empty_like(a)
        nn.conv3x3(xs, wt, bias, n, cin, cout, h, w, z=z, a=a)
        # the data gradient of a layer from cout to cin channels: x is its dz
        nn.conv3x3_dgrad_relu(xs, None, wt, act, dza, n, cout, cin, h, w)
        torch.cuda.synchronize()
        out.append((z.cpu(), a.cpu(), dza.cpu()))
    assert all(torch.equal(p, q) for p, q in zip(*out))


# few channels, single rows and columns, tiny images: either side of the rule between
# the two kernels for any shape
@pytest.mark.parametrize("n,cin,cout,h,w", [(8, 3, 16, 64, 65), (8, 1, 128, 30, 31), (4, 2, 70, 33, 65), (2, 17, 65, 1, 200),
                                             (2, 40, 33, 200, 1), (64, 8, 8, 2, 100), (3, 12, 96, 40, 41), (300, 6, 10, 1, 1),
                                             (64, 100, 20, 3, 50), (1, 384, 70, 1, 33)])
def test_both_kernels_for_any_shape(nn, n, cin, cout, h, w):  # noqa: F811
    T.test_conv_forward(nn, n, cin, cout, h, w)
    T.test_conv_backward(nn, n, cin, cout, h, w)


@pytest.mark.parametrize("n,cin,cout,h,w", [(2, 32, 32, 32, 48), (3, 64, 64, 16, 16), (1, 64, 32, 48, 32)])
def test_convolution_in_place(nn, n, cin, cout, h, w):  # noqa: F811
    """A regular convolution may write over its input: the activation over x, the FP32
    output over a buffer that x is a part of; the same bits as into other memory."""
    g = torch.Generator().manual_seed(h)
    x = T.bits(T.bf16_round(torch.randn(cin, n, h, w, generator=g))).reshape(-1)
    wt = T.bits(T.bf16_round(torch.randn(cout, 9 * cin, generator=g) / math.sqrt(9 * cin)))
    px = n * h * w
    z, a = torch.empty(cout * px, device="cuda"), torch.empty(cout * px, dtype=torch.int16, device="cuda")
    nn.conv3x3(x, wt, None, n, cin, cout, h, w, z=z, a=a)
    over = x.clone()
    nn.conv3x3(over, wt, None, n, cin, cout, h, w, a=over)
    buf = torch.empty(max(cout, cin) * px, device="cuda")  # FP32: twice the bytes of x
    part = buf.view(torch.int16)[cin * px // 2:][:cin * px]
    part.copy_(x)
    nn.conv3x3(part, wt, None, n, cin, cout, h, w, z=buf)
    torch.cuda.synchronize()
    assert torch.equal(over[:cout * px].cpu(), a.cpu())
    assert torch.equal(buf[:cout * px].cpu(), z.cpu())
    # the data gradient of a layer from cout to cin channels over its dz
    dz = torch.empty(max(cout, cin) * px, device="cuda")
    part = dz.view(torch.int16)[:cin * px]
    part.copy_(x)
    nn.conv3x3_dgrad(part, None, wt, dz, n, cout, cin, h, w)
    torch.cuda.synchronize()
    assert torch.equal(dz[:cout * px].cpu(), z.cpu())


def test_more_tiles_than_a_one_dimensional_grid_takes(nn):  # noqa: F811
    """65535 images of 128 x 136: 2^24 tiles and more.  Whole numbers, so every order of
    the sums gives the same bits: repeats of 64 images give repeats of their result."""
    n, cin, h, w, r = 65535, 4, 128, 136, 64
    if torch.cuda.mem_get_info()[0] < 20 << 30:
        pytest.skip("20 GiB of device memory")
    g = torch.Generator().manual_seed(1)
    px = h * w
    part = T.bits(torch.randint(-3, 4, (cin, r, px), generator=g).float())
    wt = T.bits(torch.randint(-2, 3, (1, 9 * cin), generator=g).float())
    want = torch.empty(r * px, dtype=torch.int16, device="cuda")
    nn.conv3x3(part, wt, None, r, cin, 1, h, w, a=want)
    x = torch.empty(cin, n, px, dtype=torch.int16, device="cuda")
    for i in range(0, n, r):
        x[:, i:i + r] = part[:, :min(r, n - i)]
    a = torch.empty(n * px, dtype=torch.int16, device="cuda")
    nn.conv3x3(x.reshape(-1), wt, None, n, cin, 1, h, w, a=a)
    torch.cuda.synchronize()
    assert int((want != 0).sum()) > 0
    for i in range(0, n, r):
        m = min(r, n - i)
        assert torch.equal(a[i * px:(i + m) * px], want[:m * px]), i
