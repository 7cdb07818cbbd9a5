"""fp32 products on the bf16 matrix instruction (every value split into three): values of all magnitudes against 64 bits, with a
bound per output, and the precision of ordinary sums."""
import numpy as np
import pytest
import torch

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl

pytestmark = pytest.mark.gpu

CASES = [
    # N, Ci, Co, H, W, ksize, stride
    (5, 16, 16, 25, 33, 3, 1),    # 3x3: two rows, one half of a stage
    (9, 48, 80, 25, 33, 3, 1),    # ... four rows, a stage and a half
    (33, 64, 64, 25, 33, 3, 1),   # ... eight rows
    (5, 20, 72, 61, 35, 3, 1),    # ... ragged channels
    (17, 40, 80, 25, 33, 3, 2),   # ... stride 2
    (2, 72, 255, 25, 33, 1, 1),   # 1x1: whole rows, an odd number of half steps
    (1, 37, 85, 25, 33, 1, 1),    # ... rows without alignment
    (1, 96, 80, 25, 33, 1, 1),    # ... whole tiles
    (5, 32, 80, 77, 95, 1, 1),    # ... buffers of 64 positions, one or two a workgroup
    (9, 64, 16, 35, 33, 1, 1),    # ... of 32, the last one with 27
    (3, 128, 80, 77, 91, 1, 1),   # ... one or two
    (3, 256, 48, 77, 91, 1, 1),
]


def run(N, Ci, Co, H, W, ks, stride, w, x, k=None):
    k = k or (9 if ks == 3 else 5)
    masks = B.rtoss_pattern_dict(k)
    idx = pl.select_patterns(w, B.F32, masks)
    y = pl.PackedLayer(Co, Ci, ks, k, B.F32, masks).pack(w, idx).conv(x, stride=stride)
    flat = w.reshape(-1).double().clone()
    G = flat.numel() // 9
    taps = torch.tensor([[int(m) >> t & 1 for t in range(9)] for m in masks], dtype=torch.float64, device="cuda")
    flat[:9 * G] *= taps[idx.long()].reshape(-1)
    flat[9 * G:] = 0
    conv = lambda a, b: torch.nn.functional.conv2d(a.permute(0, 3, 1, 2).cpu(), b.cpu(), stride=stride, padding=ks // 2).permute(0, 2, 3, 1)
    wd, xd = flat.reshape(w.shape), x.double()
    return y.double().cpu(), conv(xd, wd), conv(xd.abs(), wd.abs())


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("spread", [0, 30, 60])
def test_bound_per_output(case, spread):
    """Magnitudes over 2^-spread .. 2^spread.  Dropped products: 2^-22 of |w x| at most (m < 2^-7, l < 2^-16 of their value); the
    accumulators round at most four times per instruction, 2^-24 of the sum of magnitudes each; two additions more."""
    N, Ci, Co, H, W, ks, stride = case
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci + Co + spread)
    def values(*shape):
        v = torch.randn(shape, generator=g, device="cuda")
        return v * torch.exp2((torch.rand(shape, generator=g, device="cuda") * 2 - 1) * spread)
    got, want, size = run(*case, values(Co, Ci, ks, ks), values(N, H, W, Ci))
    steps = -(-Ci // 32) * ks * ks
    assert bool(((got - want).abs() <= size * (2.0 ** -22 + (4 * steps + 2) * 2.0 ** -24)).all())


@pytest.mark.parametrize("case", CASES)
def test_ordinary_sums_are_as_precise_as_the_fp32_instruction(case):
    """2-norm over 2-norm, no more than what v_mfma_f32_16x16x4_f32 measures: 1.04e-8 sqrt(K) for K random products of a sum
    (2.5e-7 at 576), a rounding per four channels.  Here the roundings are at most half as many: K = 32 at a time, and one or two
    an instruction, of which a stage with 16 channels has as many as one with 32."""
    N, Ci, Co, H, W, ks, stride = case
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci * Co)
    got, want, _ = run(*case, torch.randn((Co, Ci, ks, ks), generator=g, device="cuda"), torch.randn((N, H, W, Ci), generator=g, device="cuda"))
    assert float((got - want).norm() / want.norm()) <= 1.04e-8 * np.sqrt(Ci * ks * ks)


FEW = [
    # N, Ci, Co, H, W, ksize, stride, k: sums of few live products
    (3, 1, 80, 77, 91, 1, 1, 2),
    (3, 5, 40, 77, 91, 1, 1, 2),     # rows without alignment
    (3, 8, 255, 77, 91, 1, 1, 3),
    (3, 20, 80, 77, 91, 1, 1, 2),
    (1, 48, 80, 25, 33, 1, 1, 2),    # whole tiles, few positions
    (5, 32, 80, 77, 95, 1, 1, 2),    # streaming
]


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("case", FEW)
def test_short_sums_lose_one_rounding(case, relu):
    """1x1 sums of 0 to 11 live products: with eight partial products little is lost but the last addition's rounding, whose 2-norm
    over random mantissas is 2^-24 / sqrt(3) / sqrt(2) = 2.4e-8 of the result (2.5 to 2.6e-8 measured; 3.2 to 3.7e-8 with six)."""
    N, Ci, Co, H, W, ks, stride, k = case
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci * Co + k)
    x = torch.randn((N, H, W, Ci), generator=g, device="cuda")
    got, want, _ = run(*case[:7], torch.randn((Co, Ci, ks, ks), generator=g, device="cuda"), x.relu() if relu else x, k)
    assert float((got - want).norm() / want.norm()) <= 2.8e-8


@pytest.mark.parametrize("Co", [16, 80])
def test_single_products_are_rounded_correctly(Co):
    """One input channel: no output is further from its product than half a unit of its last place, 2^-24 of it, and the roundings of the
    small products, seven of 2^-24 of their accumulator (2^-6 of the product at most)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(Co)
    case = (3, 1, Co, 77, 91, 1, 1)
    got, want, size = run(*case, torch.randn((Co, 1, 1, 1), generator=g, device="cuda"), torch.randn((3, 77, 91, 1), generator=g, device="cuda"), 2)
    assert bool(((got - want).abs() <= size * 2.0 ** -24 * (1 + 7 * 2.0 ** -6)).all())


@pytest.mark.parametrize("case", CASES[:1] + CASES[-1:])
def test_largest_values_stay_finite(case):
    """The high part is truncated, so it never rounds up to infinity."""
    N, Ci, Co, H, W, ks, stride = case
    big = float(np.finfo(np.float32).max)
    w = torch.zeros((Co, Ci, ks, ks), device="cuda")
    w[:, 0, ks // 2, ks // 2] = 1.0
    x = torch.full((N, H, W, Ci), -big, device="cuda")
    got, want, _ = run(*case, w, x)
    assert torch.equal(got, want)


@pytest.mark.parametrize("case", CASES)
def test_infinite_values_give_what_an_fp32_sum_gives(case):
    """Infinities in the input, kept weights with and without bits below the first eight: the result's infinities and NaN stand
    where 64 bits has them (0 * inf under a pruned weight, sums of both signs), and the rest keeps its bound."""
    N, Ci, Co, H, W, ks, stride = case
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci - Co)
    w = torch.randn((Co, Ci, ks, ks), generator=g, device="cuda")
    w[:, ::2] = torch.where(w[:, ::2] < 0, -1.0, 1.0)
    x = torch.randn((N, H, W, Ci), generator=g, device="cuda")
    for i, value in enumerate([np.inf, -np.inf, np.nan]):
        x[0, 4 + 9 * (i % 2), 3 + 8 * i, i % Ci] = float(value)
    x[N - 1, H - 1, W - 2: W, Ci - 1] = float("inf")
    got, want, size = run(*case, w, x)
    if ks == 1:  # (groups of nine lie across the flat 1x1 weights: every pruned one under an infinite value gives NaN)
        assert bool(want.isinf().any()) and bool(want.isnan().any())
    finite = want.isfinite()
    assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got[want.isinf()], want[want.isinf()])
    steps = -(-Ci // 32) * ks * ks
    assert bool(((got - want).abs()[finite] <= (size * (2.0 ** -22 + (4 * steps + 2) * 2.0 ** -24))[finite]).all())
