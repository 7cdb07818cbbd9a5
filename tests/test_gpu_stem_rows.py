"""The image stem reads its rows as aligned words: widths and channel counts whose rows begin in the lower half of a word, the
upper one, or both in turn, at the left and right edge of the image and of a tile (32 columns), and images smaller than a tile."""
import pytest
import torch

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

from test_gpu_conv import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("Ci", [1, 2, 3])
@pytest.mark.parametrize("H,W", [(1, 1), (2, 3), (17, 64), (9, 65), (19, 66), (8, 127), (33, 34)])
def test_rows(H, W, Ci, stride):
    run_case(wl.F16 if (H + Ci) % 2 else wl.BF16, 3, Ci, 32, H, W, 3, stride, 3, False, seed=H * 100 + W + Ci)


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("Ci", [1, 2, 3])
def test_infinite_pixels(Ci, stride):
    """All nine weights live, one infinite pixel per 6x6 in turn at every place of a tile row: each output has one of them under one tap
    at most, and is infinite with that weight's sign or finite, in 64 bits and here (matrix slots past the 9 * Ci products add nothing)."""
    N, H, W, Co = 1, 36, 80, 16
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci)
    w = torch.randn((Co, Ci, 3, 3), generator=g, device="cuda").to(torch.bfloat16)
    x = torch.randn((N, H, W, Ci), generator=g, device="cuda").to(torch.bfloat16)
    for i, h in enumerate(range(stride - 1, H, 6)):
        x[0, h, i % 6::6, i % Ci] = float("inf")
    masks = B.rtoss_pattern_dict(9)
    y = pl.PackedLayer(Co, Ci, 3, 9, B.BF16, masks).pack(w, pl.select_patterns(w, B.BF16, masks)).conv(x, stride=stride, out_dt=B.F32).cpu()
    want = torch.nn.functional.conv2d(x.double().cpu().permute(0, 3, 1, 2), w.double().cpu(), stride=stride, padding=1).permute(0, 2, 3, 1)
    assert bool(want.isinf().any()) and not bool(want.isnan().any())
    assert torch.equal(y.double()[want.isinf()], want[want.isinf()]) and bool(y[want.isfinite()].isfinite().all())
