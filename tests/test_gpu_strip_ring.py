"""GPU parity of the 3x3 strips with helper waves: every height and layout, three stages (fewer than the ring has buffers) to sixteen, rows and
columns one past a tile and one short of it, padded channel blocks.  16-bit results against the fp32 ones of the kernels without helpers, which add in
the same order: the same bits once rounded.  (Against the oracle: test_gpu_variants.py.)"""
import pytest
import torch

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # rows of a wave, dt, N, Ci, Co, H, W, k
    (2, wl.F16, 1, 96, 320, 57, 79, 3),
    (2, wl.BF16, 1, 512, 256, 56, 81, 2),
    (2, wl.BF16, 1, 160, 208, 49, 97, 4),
    (3, wl.BF16, 6, 128, 240, 25, 47, 3),
    (3, wl.F16, 2, 512, 256, 61, 65, 4),
    (4, wl.F16, 4, 160, 112, 79, 95, 3),
    (4, wl.BF16, 1, 256, 512, 79, 80, 4),
    (5, wl.BF16, 1, 192, 240, 99, 161, 2),
    (5, wl.F16, 2, 96, 128, 99, 175, 4),
]


# as many tiles as the pipelined kernel takes otherwise, which computes their fp32 results: the same sums, an output stage of its own
WIDE_CASES = [
    (5, wl.F16, 15, 512, 496, 20, 19, 3),
    (5, wl.BF16, 24, 256, 272, 19, 20, 5),
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_ring_against_strips(case):
    tn, dt, N, Ci, Co, H, W, k = case
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci + H)
    T = pl.TORCH_DTYPE[dt]
    masks = B.rtoss_pattern_dict(k)
    w = (torch.randn((Co, Ci, 3, 3), generator=g, device="cuda") / Ci ** 0.5).to(T)
    layer = pl.PackedLayer(Co, Ci, 3, k, dt, masks).pack(w, pl.select_patterns(w, dt, masks))
    x = torch.randn((N, H, W, Ci), generator=g, device="cuda").to(T)
    assert torch.equal(layer.conv(x, relu=True), layer.conv(x, relu=True, out_dt=wl.F32).to(T))
    scale, bias = torch.rand(Co, generator=g, device="cuda") + 0.5, torch.randn(Co, generator=g, device="cuda")
    res = torch.randn((N, H, W, Co), generator=g, device="cuda").to(T)
    buf = torch.full((N, H, W, Co + 16), 7.0, device="cuda", dtype=T)
    layer.conv_fused(x, scale=scale, bias=bias, act=B.ACT_SILU, residual=res, y=buf[..., 8:8 + Co])
    want = layer.conv_fused(x, scale=scale, bias=bias, act=B.ACT_SILU, residual=res.float(), out_dt=wl.F32).to(T)
    assert torch.equal(buf[..., 8:8 + Co], want)
    assert bool((buf[..., :8] == 7.0).all()) and bool((buf[..., 8 + Co:] == 7.0).all())


@pytest.mark.parametrize("case", WIDE_CASES, ids=str)
def test_ring_against_the_pipelined_kernel(case):
    tn, dt, N, Ci, Co, H, W, k = case
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci + H)
    T = pl.TORCH_DTYPE[dt]
    masks = B.rtoss_pattern_dict(k)
    w = (torch.randn((Co, Ci, 3, 3), generator=g, device="cuda") / Ci ** 0.5).to(T)
    layer = pl.PackedLayer(Co, Ci, 3, k, dt, masks).pack(w, pl.select_patterns(w, dt, masks))
    x = torch.randn((N, H, W, Ci), generator=g, device="cuda").to(T)
    assert torch.equal(layer.conv(x, relu=True), layer.conv(x, relu=True, out_dt=wl.F32).to(T))
    stage = dict(scale=torch.rand(Co, generator=g, device="cuda") + 0.5, bias=torch.randn(Co, generator=g, device="cuda"), act=B.ACT_SILU)
    want = layer.conv_fused(x, out_dt=wl.F32, **stage)
    # one rounding to the stored type (half a unit), and the fp32 roundings of two orders of one output stage
    bound = want.abs() * {wl.F16: 2.0 ** -11, wl.BF16: 2.0 ** -8}[dt] + 1e-5 * want.abs().max()
    assert ((layer.conv_fused(x, **stage).float() - want).abs() <= bound).all()
