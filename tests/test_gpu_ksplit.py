"""GPU parity of the 3x3 kernel that splits the input channels over the waves of a workgroup (launches too small to fill
the chip): every tile variant of every tap layout, stage counts below, at and above the four waves, edges of tiles."""
import numpy as np
import pytest
import torch

import oracle
from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

from gpu_util import GpuLayer
from test_gpu_conv import check, run_case

pytestmark = pytest.mark.gpu

CASES = [
    # dt, N, Ci, Co,  H,  W, stride, k
    (wl.F16, 1, 32, 16, 1, 1, 1, 3),        # 16 channels x 4x8 positions: one stage, one position
    (wl.BF16, 1, 96, 48, 5, 9, 1, 3),       # ... three stages, one row and column past a tile
    (wl.F16, 2, 160, 144, 8, 8, 1, 2),      # ... five stages, whole tiles, padded channel tiles
    (wl.BF16, 1, 256, 256, 13, 21, 1, 3),
    (wl.F16, 1, 256, 240, 25, 42, 1, 3),    # 32 channels x 4x8
    (wl.BF16, 2, 64, 80, 43, 57, 1, 2),
    (wl.F16, 1, 128, 128, 60, 76, 1, 3),    # 32 channels x 8x8
    (wl.BF16, 1, 128, 256, 37, 39, 2, 3),   # stride 2: 32 channels x 4x4
    (wl.F16, 1, 32, 64, 28, 41, 2, 2),
    (wl.F16, 1, 128, 256, 61, 79, 2, 2),    # stride 2: 64 channels x 4x8
    (wl.F16, 1, 128, 112, 19, 23, 1, 4),    # three tap groups
    (wl.BF16, 1, 64, 64, 40, 50, 1, 4),
    (wl.F16, 1, 64, 64, 57, 70, 1, 4),
    (wl.F16, 1, 96, 160, 21, 23, 2, 4),
    (wl.BF16, 1, 128, 256, 56, 58, 2, 4),
    (wl.F16, 1, 256, 128, 20, 21, 1, 5),    # ... with taps in their second group
    (wl.BF16, 1, 64, 96, 27, 30, 2, 5),
    (wl.F16, 2, 128, 160, 33, 35, 2, 5),
    (wl.F16, 1, 256, 128, 20, 21, 1, 6),    # one dense step per tap
    (wl.BF16, 1, 64, 96, 27, 30, 2, 6),
    (wl.F16, 2, 128, 160, 33, 35, 2, 6),
    (wl.F32, 1, 64, 64, 23, 26, 1, 3),      # fp32
    (wl.F32, 1, 80, 48, 11, 9, 1, 4),
    (wl.F32, 1, 64, 64, 31, 33, 2, 3),
    (wl.F32, 2, 32, 144, 30, 41, 2, 2),
]


@pytest.mark.parametrize("case", CASES)
def test_channel_split_variants(case):
    dt, N, Ci, Co, H, W, stride, k = case
    run_case(dt, N, Ci, Co, H, W, 3, stride, k, relu=bool(Ci & 32), seed=Ci + Co + H, w_std=0.02)


@pytest.mark.parametrize("dt,N,Ci,Co,H,W,stride,k", [(wl.F16, 1, 96, 96, 9, 11, 1, 3), (wl.BF16, 1, 64, 64, 41, 50, 1, 3),
                                                     (wl.F16, 1, 64, 128, 21, 23, 2, 3), (wl.F32, 1, 64, 32, 9, 12, 1, 3)])
def test_channel_split_output_stage(dt, N, Ci, Co, H, W, stride, k):
    """Scale, bias, SiLU and a shortcut, written into a channel slice."""
    rng = np.random.default_rng(Ci * Co)
    masks = B.rtoss_pattern_dict(k)
    xs = wl.round_to_dtype(rng.standard_normal((N, Ci, H, W)), dt)
    ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, 3, 3)) * 0.05, dt)
    scale, bias = rng.uniform(0.5, 1.5, Co).astype(np.float32), rng.standard_normal(Co).astype(np.float32)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    res = rng.standard_normal((N, Ho, Wo, Co)).astype(np.float32)
    g = GpuLayer(ws, dt, masks, k)
    buf = torch.full((N, Ho, Wo, Co + 32), 7.0, device="cuda")
    g.layer.conv_fused(pl.to_device(wl.nchw_to_nhwc(xs), dt), stride=stride, scale=torch.from_numpy(scale).cuda(),
                       bias=torch.from_numpy(bias).cuda(), act=B.ACT_SILU, residual=torch.from_numpy(res).cuda(), out_dt=wl.F32,
                       y=buf[..., 16:16 + Co])
    torch.cuda.synchronize()
    out = buf.cpu().numpy()
    want = oracle.conv2d_fused(wl.to_f64(xs, dt), oracle.mask(wl.to_f64(ws, dt), masks, g.idx_host()), stride, scale=scale, bias=bias,
                               act=B.ACT_SILU, residual=wl.nhwc_to_nchw(res).astype(np.float64))
    check(wl.nhwc_to_nchw(out[..., 16:16 + Co]), want, dt)
    assert (out[..., :16] == 7.0).all() and (out[..., 16 + Co:] == 7.0).all()


@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("dt,N,Ci,Co,H,W,k", [
    (wl.F16, 1, 32, 16, 1, 1, 3),      # 16 channels x 4x8 positions: one stage, one position
    (wl.BF16, 1, 160, 144, 9, 17, 2),  # ... five stages, an unpaired channel block
    (wl.F16, 2, 96, 80, 31, 33, 5),    # 32 channels x 4x8, more steps than LDS holds at a time
    (wl.BF16, 1, 128, 128, 62, 81, 3),  # ... more than one round of workgroups
    (wl.F16, 1, 64, 64, 90, 121, 3),   # 32 channels x 8x8
])
def test_channel_split_of_block_shared_patterns(dt, N, Ci, Co, H, W, k, shared):
    rng = np.random.default_rng(Ci + H + k)
    masks = B.rtoss_pattern_dict(k)
    xs = wl.round_to_dtype(rng.standard_normal((N, Ci, H, W)), dt)
    ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, 3, 3)) * 0.05, dt)
    idx = rng.integers(0, len(masks), (Co, Ci)).astype(np.uint8)
    if shared:
        idx[:] = np.repeat(idx[:1, ::8], 8, 1)
    ref = oracle.conv2d(wl.to_f64(xs, dt), oracle.mask(wl.to_f64(ws, dt), masks, idx.reshape(-1)), relu=True)
    lay = pl.CoherentLayer(Co, Ci, k, dt, masks).pack(pl.to_device(ws, dt), torch.from_numpy(idx.reshape(-1)).cuda())
    x = pl.to_device(wl.nchw_to_nhwc(xs), dt)
    y32, y16 = lay.conv(x, relu=True, out_dt=wl.F32), lay.conv(x, relu=True)
    torch.cuda.synchronize()
    got = wl.nhwc_to_nchw(pl.to_host(y32)).astype(np.float64)
    assert np.max(np.abs(got - ref)) <= 2e-3 * np.sqrt(np.mean(ref ** 2))
    assert np.array_equal(wl.nhwc_to_nchw(pl.to_host(y16)), wl.round_to_dtype(got, dt))
