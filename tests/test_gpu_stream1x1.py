"""GPU parity of the streaming 1x1 kernel where its helpers' turns and its output tiles can go wrong: one, two, three and more buffers
a workgroup, a last buffer that is not full, channel blocks that do not fill a tile, one helper and two, outputs into a channel
slice with a shortcut, and arguments of SiLU past the range of its reciprocal."""
import numpy as np
import pytest
import torch

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

from gpu_util import GpuLayer, decode_live_section

pytestmark = pytest.mark.gpu

CASES = [
    # dt, Ci, Co, positions
    (wl.F16, 32, 32, 1), (wl.BF16, 32, 144, 257), (wl.F16, 32, 64, 40_003), (wl.BF16, 32, 16, 200_009),
    (wl.F16, 64, 16, 63), (wl.BF16, 64, 80, 9_999), (wl.F16, 64, 256, 70_001), (wl.F16, 64, 48, 150_001),
    (wl.F16, 128, 64, 70_017), (wl.BF16, 128, 48, 150_005), (wl.F16, 128, 208, 33_333), (wl.F16, 128, 128, 65_537),
    (wl.BF16, 256, 64, 66_001), (wl.F16, 256, 112, 40_007), (wl.F16, 256, 320, 30_011),
    (wl.F16, 512, 32, 40_009), (wl.BF16, 512, 176, 12_345), (wl.F16, 512, 256, 6_401), (wl.F16, 512, 256, 20_011),
    (wl.F16, 1024, 64, 20_003), (wl.BF16, 1024, 272, 7_001),
    (wl.F32, 16, 48, 40_003), (wl.F32, 512, 80, 20_003), (wl.F32, 64, 48, 40_001), (wl.F32, 256, 64, 20_001),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "dt%d_%d-%d_%d" % c)
def test_streaming_1x1(case):
    dt, Ci, Co, P = case
    rng = np.random.default_rng(Ci * Co + P)
    masks, k = B.rtoss_pattern_dict(2), 2
    layer = GpuLayer(wl.round_to_dtype(rng.standard_normal((Co, Ci, 1, 1)) / np.sqrt(Ci / 4), dt), dt, masks, k)
    w = wl.to_f64(decode_live_section(layer.blob_host(), Co, Ci, 1, k, dt, masks)[0], dt).reshape(Co, Ci)
    g = torch.Generator(device="cuda")
    g.manual_seed(P)
    T = pl.TORCH_DTYPE[dt]
    x = torch.randn((1, 1, P, Ci), generator=g, device="cuda").to(T)
    scale = torch.rand(Co, generator=g, device="cuda") + 0.5
    scale[::5] *= 60.0  # some arguments beyond +-80
    bias = torch.randn(Co, generator=g, device="cuda")
    shortcut = torch.randn((1, 1, P, Co + 16), generator=g, device="cuda")
    conv = x.double().reshape(P, Ci) @ torch.from_numpy(w).cuda().t()
    u = conv * scale.double() + bias.double()
    # fp32 sums of at most Ci products of unit size, relative to the largest value (the slope of SiLU is at most 1.1)
    err = 1.1e-5 * float(u.abs().max())
    for out_dt, eps in ((wl.F32, 1e-6), (dt, {wl.F32: 1e-6, wl.F16: 2.0 ** -11, wl.BF16: 2.0 ** -8}[dt])):
        To = pl.TORCH_DTYPE[out_dt]
        plain = layer.layer.conv(x, out_dt=out_dt).double().reshape(P, Co)
        assert ((plain - conv).abs() <= 1e-5 * float(conv.abs().max()) + eps * conv.abs()).all()
        buf = torch.full((1, 1, P, Co + 24), 7.0, device="cuda", dtype=To)
        for act, want in ((B.ACT_SILU, u / (1 + torch.exp(-u))), (B.ACT_RELU, u.clamp(min=0))):
            res = shortcut.to(To)[..., 8:8 + Co] if act == B.ACT_SILU else None
            if res is not None:
                want = want + res.double().reshape(P, Co)
            layer.layer.conv_fused(x, scale=scale, bias=bias, act=act, residual=res, out_dt=out_dt, y=buf[..., 8:8 + Co])
            got = buf.double().reshape(P, Co + 24)
            assert ((got[:, 8:8 + Co] - want).abs() <= err + 2 * eps * want.abs()).all()
            assert (got[:, :8] == 7.0).all() and (got[:, 8 + Co:] == 7.0).all()
