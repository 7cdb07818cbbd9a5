"""GPU parity of the 3x3 kernel over strips of output rows: every strip height and buffering of every tap layout, rows and
columns one past a tile, padded channel blocks, the fused output stage into a channel slice.  Sampled against the oracle
(the launches that belong to this kernel are too large for its full convolution)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

from gpu_util import GpuLayer

pytestmark = pytest.mark.gpu

CASES = [
    # dt, N, Ci, Co,  H,  W, k
    (wl.F16, 2, 32, 64, 101, 97, 3),     # one stage
    (wl.BF16, 1, 64, 80, 111, 113, 3),   # two rows per wave, two buffers; padded channel block
    (wl.F16, 4, 96, 128, 61, 65, 2),     # three rows per wave, two buffers, once over the chip
    (wl.BF16, 2, 64, 256, 97, 81, 3),    # ... twice
    (wl.F16, 16, 64, 64, 81, 79, 3),     # four rows per wave
    (wl.BF16, 3, 64, 64, 65, 81, 4),     # three tap groups: two, ...
    (wl.F16, 4, 64, 256, 49, 65, 4),     # ... three,
    (wl.F16, 4, 64, 128, 99, 129, 4),    # ... four,
    (wl.BF16, 2, 64, 256, 99, 161, 4),   # ... five rows per wave
    (wl.F16, 4, 64, 64, 79, 80, 5),      # dense mode: weights past LDS, eight rows
    (wl.BF16, 3, 64, 112, 81, 97, 5),    # three groups, taps in the second of theirs: two rows per wave,
    (wl.F16, 4, 64, 256, 49, 65, 5),     # ... three,
    (wl.BF16, 4, 64, 128, 99, 129, 5),   # ... four,
    (wl.F16, 2, 64, 256, 100, 167, 5),   # ... five
    (wl.BF16, 3, 64, 112, 81, 97, 6),    # dense mode, weights through LDS: two,
    (wl.F16, 4, 64, 256, 49, 65, 6),     # ... three,
    (wl.BF16, 4, 64, 128, 99, 129, 6),   # ... four,
    (wl.F16, 2, 64, 256, 100, 167, 6),   # ... five
    (wl.F32, 4, 32, 256, 59, 65, 3),     # fp32: five rows per wave
    (wl.F32, 2, 48, 208, 99, 97, 4),
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("fused", [False, True])
def test_strip_variants(case, fused):
    dt, N, Ci, Co, H, W, k = case
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci + Co + H)
    rng = np.random.default_rng(Ci * 3 + Co + H)
    masks = B.rtoss_pattern_dict(k)
    ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, 3, 3)) * 0.05, dt)
    layer = GpuLayer(ws, dt, masks, k)
    T = pl.TORCH_DTYPE[dt]
    x = torch.randn((N, H, W, Ci), generator=g, device="cuda").to(T)
    extra = {}
    if fused:
        scale, bias = torch.rand(Co, generator=g, device="cuda") + 0.5, torch.randn(Co, generator=g, device="cuda")
        res = torch.randn((N, H, W, Co), generator=g, device="cuda")
        buf = torch.full((N, H, W, Co + 16), 7.0, device="cuda")
        layer.layer.conv_fused(x, scale=scale, bias=bias, act=B.ACT_SILU, residual=res, out_dt=wl.F32, y=buf[..., 8:8 + Co])
        y = buf[..., 8:8 + Co]
        assert bool((buf[..., :8] == 7.0).all()) and bool((buf[..., 8 + Co:] == 7.0).all())
        extra = dict(scale=scale.cpu().numpy(), bias=bias.cpu().numpy(), act=B.ACT_SILU)
    else:
        y = layer.layer.conv(x, relu=True, out_dt=wl.F32)
        if dt != wl.F32:
            assert torch.equal(layer.layer.conv(x, relu=True), y.to(T))
    pruned = oracle.mask(wl.to_f64(ws, dt), masks, layer.idx_host())
    # windows of the image with their halo: corners, the last rows and columns, a seam between tiles
    err, ref2, cnt, ref_max = 0.0, 0.0, 0, 0.0
    for n in (0, N - 1):
        for h0, w0 in ((0, 0), (H - 7, W - 9), (max(0, H // 2 - 3), max(0, W // 2 - 3)), (0, W - 9)):
            h1, w1 = min(h0 + 7, H), min(w0 + 9, W)
            top, left = int(h0 > 0), int(w0 > 0)
            xin = x[n:n + 1, h0 - top: min(h1 + 1, H), w0 - left: min(w1 + 1, W)].double().cpu().numpy()
            xin = wl.nhwc_to_nchw(xin)
            if fused:
                r = np.zeros((1, Co) + xin.shape[2:])
                r[:, :, top:top + h1 - h0, left:left + w1 - w0] = wl.nhwc_to_nchw(res[n:n + 1, h0:h1, w0:w1].double().cpu().numpy())
                ref = oracle.conv2d_fused(xin, pruned, 1, residual=r, **extra)
            else:
                ref = oracle.conv2d(xin, pruned, relu=True)
            ref = ref[:, :, top:top + h1 - h0, left:left + w1 - w0]
            got = wl.nhwc_to_nchw(y[n:n + 1, h0:h1, w0:w1].double().cpu().numpy())
            err, ref_max = max(err, np.max(np.abs(got - ref))), max(ref_max, np.max(np.abs(ref)))
            ref2, cnt = ref2 + np.sum(ref ** 2), cnt + ref.size
    assert err <= (1e-5 * ref_max if dt == wl.F32 else 2e-3 * np.sqrt(ref2 / cnt))
