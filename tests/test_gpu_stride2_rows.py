"""GPU parity of the stride-2 kernels where their stores can go wrong: pairs of columns of which one is outside the image, rows of
channels that end within a block of 64, one and two blocks of positions a wave, outputs into a channel slice with a shortcut."""
import numpy as np
import pytest
import torch

import oracle
from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

from gpu_util import GpuLayer

pytestmark = pytest.mark.gpu

# dt, k, N, Ci, Co, H, W: the single-buffered kernel's, and the resident one's (images of one block, several channel blocks, a last turn of few blocks)
CASES = [(wl.F16, 3, 17, 32, 16, 18, 17), (wl.BF16, 2, 520, 64, 112, 1, 1), (wl.F16, 2, 40, 32, 48, 5, 31), (wl.BF16, 4, 9, 32, 80, 33, 35),
         (wl.F16, 3, 40, 128, 272, 42, 41), (wl.F16, 5, 12, 64, 80, 45, 43), (wl.BF16, 5, 65, 96, 80, 41, 29)]
RESIDENT_CASES = [(wl.F16, 3, 17, 32, 16, 107, 109), (wl.BF16, 2, 10, 64, 144, 79, 85), (wl.F16, 2, 100, 32, 80, 5, 140),
                  (wl.BF16, 3, 3201, 64, 64, 1, 1), (wl.F16, 3, 9, 64, 320, 66, 67)]


@pytest.mark.parametrize("case", CASES + RESIDENT_CASES, ids=lambda c: "-".join(map(str, c)))
def test_stride_2_rows(case):
    dt, k, N, Ci, Co, H, W = case
    rng = np.random.default_rng(Ci + Co + W)
    masks = B.rtoss_pattern_dict(k)
    ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, 3, 3)) / np.sqrt(Ci * k), dt)
    xs = wl.round_to_dtype(rng.standard_normal((N, Ci, H, W)), dt)
    g = GpuLayer(ws, dt, masks, k)
    wv = wl.to_f64(ws, dt)
    conv = oracle.conv2d(wl.to_f64(xs, dt), oracle.mask(wv, masks, oracle.select(wv, masks)), stride=2).transpose(0, 2, 3, 1)
    scale, bias = rng.random(Co).astype(np.float32) + 0.5, rng.standard_normal(Co).astype(np.float32)
    u = conv * scale + bias
    x, T = pl.to_device(wl.nchw_to_nhwc(xs), dt), pl.TORCH_DTYPE[dt]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(W)
    shortcut = torch.randn(conv.shape[:3] + (Co + 16,), generator=gen, device="cuda").to(T)[..., 8:8 + Co]
    buf = torch.full(conv.shape[:3] + (Co + 24,), 7.0, device="cuda", dtype=T)
    g.layer.conv_fused(x, stride=2, scale=torch.from_numpy(scale).cuda(), bias=torch.from_numpy(bias).cuda(), act=B.ACT_SILU,
                       residual=shortcut, y=buf[..., 8:8 + Co])
    want = u / (1 + np.exp(-u)) + shortcut.double().cpu().numpy()
    got = buf.double().cpu().numpy()
    # fp32 sums of at most Ci * k products relative to the largest value (the slope of SiLU is at most 1.1), and one rounding
    bound = 1.1e-5 * np.abs(u).max() + (2.0 ** -11 if dt == wl.F16 else 2.0 ** -8) * np.abs(want)
    assert (np.abs(got[..., 8:8 + Co] - want) <= bound).all()
    assert (got[..., :8] == 7.0).all() and (got[..., 8 + Co:] == 7.0).all()
    plain = g.layer.conv(x, stride=2)
    assert (np.abs(plain.double().cpu().numpy() - conv) <= 1e-5 * np.abs(conv).max() + (2.0 ** -11 if dt == wl.F16 else 2.0 ** -8) * np.abs(conv)).all()
