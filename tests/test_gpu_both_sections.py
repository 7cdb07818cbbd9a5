"""GPU parity of layers whose dictionary needs repeated taps (5 entries): the weights are packed as 2-of-4 and as dense fragments, and a launch reads
the section that is faster.  One layer on shapes of either route, channel tiles padded differently in the two, every pattern; against
64-bit sums of the same pruned weights (an fp32 sum of Ci * k products of normal values differs from them by at most 1e-5 of the largest)."""
import pytest
import torch

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

from test_gpu_rows_groups import reference

pytestmark = pytest.mark.gpu

# section, stride, launches (N, Ci, Co, H, W)
ROUTES = [
    ("dense", 1, [(2, 96, 144, 17, 33), (2, 64, 80, 29, 35), (1, 256, 256, 20, 46), (3, 128, 128, 32, 48), (200, 192, 160, 7, 6), (41, 96, 256, 23, 17)]),
    ("2-of-4", 1, [(1, 96, 144, 17, 33), (2, 64, 80, 9, 19), (1, 512, 80, 41, 43), (9, 96, 240, 7, 33), (1, 256, 256, 49, 83), (2, 96, 208, 99, 161),
                   (16, 128, 256, 39, 41), (5, 64, 96, 81, 79)]),
    ("dense", 2, [(1, 96, 144, 61, 129), (1, 224, 448, 33, 57)]),
    ("2-of-4", 2, [(1, 96, 144, 11, 13), (2, 64, 144, 21, 67), (4, 64, 128, 101, 135), (3, 192, 400, 71, 91), (65, 96, 80, 41, 29)]),
]
LAYERS = sorted({(Ci, Co) for _, _, shapes in ROUTES for _, Ci, Co, _, _ in shapes})


@pytest.mark.parametrize("dt", [wl.F16, wl.BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("Ci,Co", LAYERS)
def test_both_sections(Ci, Co, dt):
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci + Co)
    T = pl.TORCH_DTYPE[dt]
    masks = B.rtoss_pattern_dict(5)
    w = (torch.randn((Co, Ci, 3, 3), generator=g, device="cuda") / Ci ** 0.5).to(T)
    idx = torch.randint(len(masks), (Co * Ci,), generator=g, device="cuda").to(torch.uint8)
    layer = pl.PackedLayer(Co, Ci, 3, 5, dt, masks)
    layer.blob.fill_(0x7f)  # (what the packer leaves out would be far off)
    layer.pack(w, idx)
    for section, stride, shapes in ROUTES:
        for N, ci, co, H, W in shapes:
            if (ci, co) != (Ci, Co):
                continue
            x = torch.randn((N, H, W, Ci), generator=g, device="cuda").to(T)
            want = reference(x, w, masks, idx)[:, ::stride, ::stride]
            y = layer.conv(x, stride=stride, out_dt=wl.F32)
            assert float((y - want).abs().max()) <= 1e-5 * float(want.abs().max()), (section, N, H, W)
            assert torch.equal(layer.conv(x, stride=stride, relu=True), y.clamp(min=0).to(T))
            buf = torch.full(y.shape[:3] + (Co + 40,), 7.0, device="cuda", dtype=T)
            layer.conv_fused(x, stride=stride, y=buf[..., 8:8 + Co])
            assert torch.equal(buf[..., 8:8 + Co], y.to(T)) and bool((buf[..., :8] == 7.0).all()) and bool((buf[..., 8 + Co:] == 7.0).all())
