"""The scalar head at image sizes around its lane layout (a power of two of lanes per
channel, up to 64) and at more images than a launch has workgroups."""
import pytest
import torch

import test_gpu_nn as T
from test_gpu_nn import nn  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c,hw", [(3, 5, 1), (700, 64, 1), (4, 3, 2), (5, 17, 9), (2, 256, 31), (3, 40, 33),
                                     (2, 16, 64), (2, 7, 65), (3, 256, 169), (3000000, 2, 1)])
def test_gap_linear(nn, n, c, hw):  # noqa: F811
    """FP64 sums: half a unit in the last place of the exact value, and 2^-45 of the sum of
    magnitudes for the FP64 sums themselves."""
    g = torch.Generator().manual_seed(c)
    a = T.bf16_round(torch.randn(c, n, hw, generator=g))
    wl, bl = torch.randn(c, generator=g), torch.randn(1, generator=g)
    out = torch.full((n,), float("nan"), device="cuda")
    nn.gap_linear(T.bits(a), wl.cuda(), bl.cuda(), out, n, c, hw)
    torch.cuda.synchronize()
    want = torch.einsum("c,cnp->n", wl.double(), a.double()) / hw + bl.double()
    mag = torch.einsum("c,cnp->n", wl.double().abs(), a.double().abs()) / hw + bl.double().abs()
    ulp = 2.0 ** (torch.floor(torch.log2(want.abs().clamp_min(1e-30))) - 23)
    assert ((out.cpu().double() - want).abs() <= 0.5 * ulp + 2.0 ** -45 * mag).all()


# 64 to 255 pixels (four channels at a time: fewer and more than the wavefronts hold),
# 256 and more, each with few images and beyond 512
@pytest.mark.parametrize("n,c,hw", [(513, 3, 64), (600, 70, 100), (520, 64, 255), (2, 200, 130), (513, 13, 256),
                                     (600, 65, 300)])
def test_gap_linear_of_many_images(nn, n, c, hw):  # noqa: F811
    test_gap_linear(nn, n, c, hw)
