"""GPU parity of the matrix-core kernels at channel counts between their stages (in) and tiles (out), and of fp32 1x1
layers: last stages with few channels, rows that are 16-, 8- and 4-byte aligned, output rows without any alignment."""
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
    # N, Ci, Co,  H,  W, ks, stride, k, relu
    (2, 24, 36, 13, 17, 3, 1, 2, True),    # a single partial stage
    (1, 40, 85, 19, 21, 3, 1, 3, False),   # a whole stage and a partial one; unaligned rows out
    (2, 48, 72, 21, 18, 3, 2, 2, False),
    (1, 80, 64, 9, 33, 3, 1, 4, True),     # three tap groups
    (1, 72, 17, 11, 12, 3, 2, 4, False),
    (1, 40, 20, 10, 10, 3, 1, 5, False),   # dense mode
    (1, 104, 255, 14, 15, 3, 2, 5, True),
    (3, 36, 255, 20, 23, 1, 1, 2, False),  # 4-byte copies of 16-bit rows
    (1, 2, 4, 7, 9, 1, 1, 3, False),
    (1, 70, 33, 12, 11, 1, 1, 3, True),
    (2, 72, 36, 25, 19, 1, 1, 2, True),    # 16-byte copies, partial stage
    (1, 264, 120, 11, 12, 1, 1, 3, False),
    (1, 192, 130, 16, 17, 1, 1, 2, False),  # whole stages, ragged channels out
    (2, 48, 144, 9, 15, 1, 1, 2, False),   # ragged in, whole tiles out
]


@pytest.mark.parametrize("dt", [wl.F32, wl.F16, wl.BF16])
@pytest.mark.parametrize("case", CASES)
def test_ragged_channel_counts(dt, case):
    N, Ci, Co, H, W, ks, stride, k, relu = case
    run_case(dt, N, Ci, Co, H, W, ks, stride, k, relu, seed=Ci * 7 + Co + dt)


FP32_1X1 = [
    # Ci = 16 * 2^n up to 512 (streaming kernel, from 64 on the channel split at these sizes): N, Ci, Co, H, W, k, relu
    (1, 16, 16, 1, 1, 2, False),
    (2, 32, 48, 11, 12, 3, True),
    (1, 64, 128, 33, 31, 2, False),
    (4, 128, 64, 40, 37, 3, False),
    (2, 256, 272, 13, 19, 2, True),
    (1, 512, 80, 9, 14, 2, False),
    (1, 1024, 32, 7, 9, 2, False),  # deeper: ring kernel
]


@pytest.mark.parametrize("case", FP32_1X1)
def test_fp32_1x1_matrix_core(case):
    N, Ci, Co, H, W, k, relu = case
    run_case(wl.F32, N, Ci, Co, H, W, 1, 1, k, relu, seed=Ci + Co, w_std=0.03)


@pytest.mark.parametrize("dt,ks,Ci,Co", [(wl.F16, 3, 40, 36), (wl.BF16, 1, 36, 85), (wl.F32, 3, 24, 20), (wl.F32, 1, 20, 33),
                                         (wl.F16, 1, 72, 72)])
def test_ragged_output_stage_writes_its_slice_only(dt, ks, Ci, Co):
    """Scale, bias, SiLU, shortcut, into a channel slice of a wider buffer whose other channels stay as they were."""
    k, N, H, W = 2, 2, 9, 14
    rng = np.random.default_rng(Ci + Co)
    masks = B.rtoss_pattern_dict(k)
    xs = wl.round_to_dtype(rng.standard_normal((N, Ci, H, W)), dt)
    ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, ks, ks)) * 0.1, dt)
    scale, bias = rng.uniform(0.5, 1.5, Co).astype(np.float32), rng.standard_normal(Co).astype(np.float32)
    g = GpuLayer(ws, dt, masks, k)
    wide = -(-Co // 8) * 8 + 16
    res = wl.round_to_dtype(rng.standard_normal((N, H, W, wide)), wl.F32)
    buf = torch.full((N, H, W, wide), 7.0, device="cuda")
    residual = torch.from_numpy(res).cuda()
    g.layer.conv_fused(pl.to_device(wl.nchw_to_nhwc(xs), dt), scale=torch.from_numpy(scale).cuda(), bias=torch.from_numpy(bias).cuda(),
                       act=B.ACT_SILU, residual=residual[..., 8:8 + Co], out_dt=wl.F32, y=buf[..., 8:8 + Co])
    torch.cuda.synchronize()
    out = buf.cpu().numpy()
    want = oracle.conv2d_fused(wl.to_f64(xs, dt), oracle.mask(wl.to_f64(ws, dt), masks, g.idx_host()), 1, scale=scale, bias=bias,
                               act=B.ACT_SILU, residual=wl.nhwc_to_nchw(res[..., 8:8 + Co]).astype(np.float64))
    check(wl.nhwc_to_nchw(out[..., 8:8 + Co]), want, dt)
    assert (out[..., :8] == 7.0).all() and (out[..., 8 + Co:] == 7.0).all()
