"""The weight and bias gradients of convolution layers whose images do not fill the
kernel's pixel tiles or whose tensors are not 16-byte aligned."""
import math

import pytest
import torch
import torch.nn.functional as Fn

import test_gpu_nn as T
from test_gpu_nn import nn  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def wgrad(nn, x, dz, n, cin, cout, h, w, shift=0, joined=False):  # noqa: F811
    m = cout * cin * 9
    g = torch.full((m + cout,), float("nan"), device="cuda")
    dw, db = (g[:m], g[m:]) if joined else (torch.empty(m, device="cuda"), torch.empty(cout, device="cuda"))
    work = torch.full((nn.wgrad_work(n, cin, cout, h, w) + 3,), float("nan"), device="cuda")
    xb, db16 = T.bits(T.to_cn(x)).reshape(-1), T.bits(T.to_cn(dz)).reshape(-1)
    if shift:
        buf = torch.zeros(db16.numel() + shift, dtype=torch.int16, device="cuda")
        buf[shift:] = db16
        db16 = buf[shift:]
    need = nn.wgrad_work(n, cin, cout, h, w)
    nn.conv3x3_wgrad(xb, db16, dw, db, work[:need], n, cin, cout, h, w)
    torch.cuda.synchronize()
    assert torch.isnan(work[need:]).all()  # nothing beyond the workspace
    return T.from_krsc(dw.cpu(), cout, cin), db.cpu()


# ragged images, several ranges of pixels, one pixel, rows below 8 pixels, many
# small images; a regular shape whose dz is one element off a 16-byte address
@pytest.mark.parametrize("n,cin,cout,h,w,shift", [
    (4, 48, 80, 50, 75, 0), (9, 3, 5, 40, 40, 0), (2, 20, 36, 13, 19, 0), (1, 2, 1, 1, 1, 0), (600, 8, 24, 3, 3, 0),
    (2, 4, 6, 333, 517, 0), (5, 1, 40, 9, 70, 0), (5, 32, 16, 32, 32, 1), (3, 64, 70, 32, 16, 1), (1, 9, 7, 1, 900, 0)])
@pytest.mark.parametrize("joined", [False, True])
def test_bias_gradient_is_rounded_once(nn, n, cin, cout, h, w, shift, joined):  # noqa: F811
    """db is the sum over all pixels in FP64, rounded once: half a unit in the last
    place of the exact sum (and the FP64 sum's own error, 2^-40 of the sum of
    magnitudes at most)."""
    g = torch.Generator().manual_seed(n + cout)
    x = T.bf16_round(torch.randn(n, cin, h, w, generator=g))
    dz = T.bf16_round(torch.randn(n, cout, h, w, generator=g) * 10 ** torch.linspace(-2, 2, h)[:, None])
    _, db = wgrad(nn, x, dz, n, cin, cout, h, w, shift, joined)
    for c in range(cout):
        v = dz[:, c].double().reshape(-1)
        want = math.fsum(v.tolist())
        ulp = 2.0 ** (math.floor(math.log2(max(abs(want), 1e-30))) - 23)
        assert abs(db[c].item() - want) <= 0.5 * ulp + 2.0 ** -40 * v.abs().sum().item(), (c, db[c].item(), want)


@pytest.mark.parametrize("n,cin,cout,h,w", [(2, 20, 36, 13, 19), (1, 40, 33, 9, 17), (3, 5, 6, 5, 7), (2, 33, 20, 1, 40)])
@pytest.mark.parametrize("where", ["corner", "right", "bottom"])
def test_infinities_stay_in_their_own_sums(nn, n, cin, cout, h, w, where):  # noqa: F811
    """An infinite input value at the last row or column of an image reaches the taps that
    multiply it by a gradient of that image, and no others (a tile hangs over the
    image there, and zero times infinity is not zero)."""
    g = torch.Generator().manual_seed(h * w)
    x = T.bf16_round(torch.randn(n, cin, h, w, generator=g))
    dz = T.bf16_round(torch.randn(n, cout, h, w, generator=g))
    y, c = {"corner": (h - 1, w - 1), "right": (h // 2, w - 1), "bottom": (h - 1, w // 2)}[where]
    x[n - 1, cin - 1, y, c] = float("inf")
    dw, db = wgrad(nn, x, dz, n, cin, cout, h, w)
    cols = Fn.unfold(x.double(), 3, padding=1)  # [n][cin 9][h w]
    want = sum(dz[k].double().reshape(cout, -1) @ cols[k].T for k in range(n)).view(cout, cin, 3, 3)
    assert torch.equal(torch.isfinite(dw), torch.isfinite(want))
    ok = torch.isfinite(want)
    sw = (dz.abs().sum() * x[torch.isfinite(x)].abs().max()).item()
    assert (dw.double() - want)[ok].abs().max().item() <= 2e-6 * sw
    assert torch.isfinite(db).all()


# at the edge of a quarter of the 8 x 16 tiles (packed pixels below): one pixel, rows,
# columns, 4 x 8 (a quarter) and one pixel less, several tiles, channels around 64
@pytest.mark.parametrize("n,cin,cout,h,w", [(1, 1, 1, 1, 1), (5, 3, 2, 1, 1), (3, 65, 63, 1, 31), (2, 17, 65, 31, 1),
                                             (4, 33, 20, 4, 8), (4, 33, 20, 1, 32), (700, 20, 64, 2, 3), (2, 64, 64, 9, 17),
                                             (40, 16, 130, 5, 5)])
def test_images_that_fill_little_of_a_tile(nn, n, cin, cout, h, w):  # noqa: F811
    """Both sides of the rule that packs the pixels of small images, with the
    tolerance of the other weight gradients."""
    g = torch.Generator().manual_seed(n + h)
    x = T.bf16_round(torch.randn(n, cin, h, w, generator=g))
    dz = T.bf16_round(torch.randn(n, cout, h, w, generator=g))
    dw, db = wgrad(nn, x, dz, n, cin, cout, h, w)
    cols = Fn.unfold(x.double(), 3, padding=1)
    want = sum(dz[k].double().reshape(cout, -1) @ cols[k].T for k in range(n)).view(cout, cin, 3, 3)
    assert (dw.double() - want).abs().max().item() <= 2e-6 * (dz.abs().sum() * x.abs().max()).item()
    assert torch.allclose(db.double(), dz.double().sum(dim=(0, 2, 3)), rtol=1e-6, atol=1e-5)
