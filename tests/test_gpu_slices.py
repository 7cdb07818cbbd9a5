"""Outputs into a channel slice of a wider buffer.  The kernels store past the L2's write-back where the slice's rows are whole
sectors of 64 bytes, and otherwise as the L2 puts them together: either way the bits of the plain call, and the other channels stay."""
import numpy as np
import pytest
import torch

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

from gpu_util import GpuLayer

pytestmark = pytest.mark.gpu

CASES = [
    # kernel, dt, N, Ci, Co, H, W, ks, stride, k
    ("conv1x1_mma", wl.F16, 1, 24, 1024, 29, 31, 1, 1, 2),  # rows of several blocks, whole sectors
    ("conv1x1_mma", wl.BF16, 1, 40, 1000, 29, 31, 1, 1, 2),  # ... not
    ("conv1x1_mma", wl.F32, 1, 24, 1000, 17, 31, 1, 1, 2),
    ("conv1x1_mma", wl.F16, 1, 24, 520, 29, 31, 1, 1, 2),
    ("conv1x1_mma", wl.F16, 1, 24, 512, 29, 31, 1, 1, 2),
    ("conv1x1_mma", wl.BF16, 1, 72, 240, 29, 31, 1, 1, 2),
    ("conv1x1_stream", wl.F16, 1, 32, 144, 29, 31, 1, 1, 2),  # straight from the accumulators
    ("conv1x1_stream", wl.BF16, 1, 64, 16, 29, 31, 1, 1, 2),
    ("conv1x1_stream", wl.F16, 1, 64, 80, 131, 129, 1, 1, 2),
    ("conv1x1_stream", wl.F16, 1, 512, 208, 83, 85, 1, 1, 2),
    ("conv1x1_stream", wl.BF16, 1, 512, 64, 151, 153, 1, 1, 2),
    ("conv3x3_strip", wl.F16, 17, 64, 128, 17, 19, 3, 1, 4),  # one buffer, two blocks of channels
    ("conv3x3_strip", wl.BF16, 49, 64, 208, 9, 19, 3, 1, 4),  # ... the last one of 16 channels
    ("conv3x3_strip", wl.F16, 33, 64, 48, 17, 19, 3, 1, 4),  # ... one block
    ("conv3x3_strip", wl.BF16, 33, 32, 48, 9, 19, 3, 1, 3),  # a single stage
    ("conv3x3_strip", wl.F16, 33, 96, 128, 16, 18, 3, 1, 5),
    ("conv3x3_strip", wl.F16, 33, 96, 128, 16, 18, 3, 1, 6),  # dense mode
    ("conv3x3_strip", wl.BF16, 97, 96, 48, 17, 18, 3, 1, 5),
    ("conv3x3_strip", wl.F16, 17, 64, 160, 9, 19, 3, 1, 3),  # two buffers
    ("conv3x3_rows", wl.BF16, 2, 128, 224, 100, 167, 3, 1, 3),
    ("conv3x3_sparse_sb", wl.F16, 9, 96, 80, 33, 35, 3, 2, 3),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_slices(case):
    kernel, dt, N, Ci, Co, H, W, ks, stride, k = case
    rng = np.random.default_rng(Ci + Co)
    layer = GpuLayer(wl.round_to_dtype(rng.standard_normal((Co, Ci, ks, ks)) / np.sqrt(Ci * k), dt), dt, B.rtoss_pattern_dict(k), k).layer
    g = torch.Generator(device="cuda")
    g.manual_seed(Co)
    x = torch.randn((N, H, W, Ci), generator=g, device="cuda").to(pl.TORCH_DTYPE[dt])
    stage = dict(scale=torch.rand(Co, generator=g, device="cuda") + 0.5, bias=torch.randn(Co, generator=g, device="cuda"), act=B.ACT_SILU)
    for out_dt in {dt, wl.F32}:
        for fused in ({}, stage):
            plain = layer.conv_fused(x, stride=stride, out_dt=out_dt, **fused)
            for first, behind in ((0, 8), (8, 8), (32, 32), (8, 56)):  # elements: rows and first element at multiples of 64 bytes or not
                pitch = -(-Co // 32) * 32 + first + behind
                buf = torch.full(plain.shape[:3] + (pitch,), 7.0, device="cuda", dtype=plain.dtype)
                layer.conv_fused(x, stride=stride, out_dt=out_dt, y=buf[..., first:first + Co], **fused)
                assert torch.equal(buf[..., first:first + Co], plain)
                assert (buf[..., :first] == 7.0).all() and (buf[..., first + Co:] == 7.0).all()
