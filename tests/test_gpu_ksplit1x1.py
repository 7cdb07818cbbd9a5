"""GPU parity of the 1x1 kernel that splits the input channels over the waves of a workgroup: every depth and tile, last
positions and channel tiles that do not fill a tile, the output stage into a channel slice."""
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
    # dt, N, Ci, Co, H, W
    (wl.F16, 1, 128, 16, 1, 1),        # 32 x 16 tiles: one position
    (wl.BF16, 1, 256, 80, 5, 7),
    (wl.F16, 1, 512, 144, 9, 13),
    (wl.F16, 2, 1024, 48, 7, 9),
    (wl.BF16, 1, 128, 256, 33, 31),    # 32 x 32
    (wl.F16, 1, 512, 512, 20, 21),
    (wl.BF16, 1, 1024, 272, 19, 23),
    (wl.F16, 2, 128, 64, 80, 79),      # 64 x 32
    (wl.BF16, 4, 256, 192, 21, 37),
    (wl.F16, 4, 512, 240, 20, 20),
    (wl.F32, 1, 64, 16, 3, 5),
    (wl.F32, 3, 64, 80, 41, 39),
    (wl.F32, 2, 128, 272, 17, 19),
    (wl.F32, 1, 256, 112, 20, 20),
    (wl.F32, 1, 512, 48, 11, 13),
]


@pytest.mark.parametrize("case", CASES)
def test_channel_split_1x1(case):
    dt, N, Ci, Co, H, W = case
    run_case(dt, N, Ci, Co, H, W, 1, 1, 2 + Co // 16 % 2, relu=Co > 100, seed=Ci + Co, w_std=0.03)


@pytest.mark.parametrize("dt,Ci,Co,H", [(wl.F16, 128, 64, 9), (wl.BF16, 512, 96, 13), (wl.F16, 1024, 32, 8), (wl.F32, 128, 48, 11)])
def test_channel_split_1x1_output_stage(dt, Ci, Co, H):
    rng = np.random.default_rng(Ci * Co)
    masks = B.rtoss_pattern_dict(2)
    xs = wl.round_to_dtype(rng.standard_normal((2, Ci, H, H)), dt)
    ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, 1, 1)) * 0.05, dt)
    scale, bias = rng.uniform(0.5, 1.5, Co).astype(np.float32), rng.standard_normal(Co).astype(np.float32)
    res = rng.standard_normal((2, H, H, Co)).astype(np.float32)
    g = GpuLayer(ws, dt, masks, 2)
    buf = torch.full((2, H, H, Co + 32), 7.0, device="cuda")
    g.layer.conv_fused(pl.to_device(wl.nchw_to_nhwc(xs), dt), scale=torch.from_numpy(scale).cuda(), bias=torch.from_numpy(bias).cuda(),
                       act=B.ACT_SILU, residual=torch.from_numpy(res).cuda(), out_dt=wl.F32, y=buf[..., 16:16 + Co])
    torch.cuda.synchronize()
    out = buf.cpu().numpy()
    want = oracle.conv2d_fused(wl.to_f64(xs, dt), oracle.mask(wl.to_f64(ws, dt), masks, g.idx_host()), 1, scale=scale, bias=bias,
                               act=B.ACT_SILU, residual=wl.nhwc_to_nchw(res).astype(np.float64))
    check(wl.nhwc_to_nchw(out[..., 16:16 + Co]), want, dt)
    assert (out[..., :16] == 7.0).all() and (out[..., 16 + Co:] == 7.0).all()
