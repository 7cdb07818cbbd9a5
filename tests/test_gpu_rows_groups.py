"""GPU parity of the pipelined 3x3 kernel on three groups of taps: tall and short tiles, rows and columns one past a tile and one short of
it, three stages (the fewest) to nine, padded channel blocks, patterns that need a tap in its second group.  Against 64-bit sums of the same
pruned weights; an fp32 sum of Ci*k products of normal values differs from them by at most 1e-5 of the largest result."""
import pytest
import torch

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # dt, N, Ci, Co, H, W, k
    (wl.BF16, 2, 96, 256, 99, 161, 5),
    (wl.F16, 1, 128, 208, 161, 159, 4),
    (wl.BF16, 70, 288, 112, 19, 31, 5),
    (wl.F16, 33, 160, 240, 37, 31, 5),
    (wl.BF16, 140, 96, 112, 20, 15, 5),
    (wl.F16, 2, 192, 448, 97, 95, 4),
]


def reference(x, w, masks, idx):
    """Shifted products in 64 bits: [N, H, W, Co]."""
    Co, Ci = w.shape[:2]
    live = torch.tensor([[m >> t & 1 for t in range(9)] for m in masks], device="cuda", dtype=torch.float64)[idx.long()]
    w = w.double() * live.reshape(w.shape)
    H, W = x.shape[1:3]
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    y = 0
    for t in range(9):
        xs = xp[:, t // 3:t // 3 + H, t % 3:t % 3 + W].reshape(-1, Ci)
        y = y + xs @ w[:, :, t // 3, t % 3].t().contiguous()
    return y.reshape(*x.shape[:3], Co)


@pytest.mark.parametrize("case", CASES, ids=str)
def test_rows_of_groups(case):
    dt, N, Ci, Co, H, W, k = case
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci + H)
    T = pl.TORCH_DTYPE[dt]
    masks = B.rtoss_pattern_dict(k)
    w = (torch.randn((Co, Ci, 3, 3), generator=g, device="cuda") / Ci ** 0.5).to(T)
    idx = torch.randint(len(masks), (Co * Ci,), generator=g, device="cuda").to(torch.uint8)  # every pattern, the rare ones too
    layer = pl.PackedLayer(Co, Ci, 3, k, dt, masks).pack(w, idx)
    x = torch.randn((N, H, W, Ci), generator=g, device="cuda").to(T)
    want = reference(x, w, masks, idx)
    y = layer.conv(x, out_dt=wl.F32)
    assert float((y - want).abs().max()) <= 1e-5 * float(want.abs().max())
    assert torch.equal(layer.conv(x, relu=True), y.clamp(min=0).to(T))
    scale, bias = torch.rand(Co, generator=g, device="cuda") + 0.5, torch.randn(Co, generator=g, device="cuda")
    res = torch.randn((N, H, W, Co), generator=g, device="cuda").to(T)
    buf = torch.full((N, H, W, Co + 16), 7.0, device="cuda", dtype=T)
    layer.conv_fused(x, scale=scale, bias=bias, act=B.ACT_SILU, residual=res, y=buf[..., 8:8 + Co])
    same = layer.conv_fused(x, scale=scale, bias=bias, act=B.ACT_SILU, residual=res.float(), out_dt=wl.F32).to(T)
    assert torch.equal(buf[..., 8:8 + Co], same)
    assert bool((buf[..., :8] == 7.0).all()) and bool((buf[..., 8 + Co:] == 7.0).all())
