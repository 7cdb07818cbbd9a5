"""The image stem reads its rows as aligned words: widths and channel counts whose rows begin in the lower half of a word, the
upper one, or both in turn, at the left and right edge of the image and of a tile (32 columns), and images smaller than a tile."""
import pytest

from paper_2303_02191_amd import workloads as wl

from test_gpu_conv import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("Ci", [1, 2, 3])
@pytest.mark.parametrize("H,W", [(1, 1), (2, 3), (17, 64), (9, 65), (19, 66), (8, 127), (33, 34)])
def test_rows(H, W, Ci, stride):
    run_case(wl.F16 if (H + Ci) % 2 else wl.BF16, 3, Ci, 32, H, W, 3, stride, 3, False, seed=H * 100 + W + Ci)
