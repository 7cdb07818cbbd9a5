"""GPU parity of every convolution kernel variant the library holds (variants.py): with and without an output stage, fp32
results against the oracle on windows of the image, 16-bit results against the fp32 ones rounded once, written into a channel
slice whose neighbours stay as they were."""
import numpy as np
import pytest
import torch

import oracle
from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

from gpu_util import GpuLayer
from test_gpu_conv import check
from variants import VARIANTS

pytestmark = pytest.mark.gpu


def windows(N, Ho, Wo):
    """Outputs to compare: whole small images, else corners, the last rows and columns and the middle, first and last image."""
    for n in sorted({0, N - 1}):
        if Ho * Wo <= 400:
            yield n, 0, Ho, 0, Wo
            continue
        for h0, w0 in {(0, 0), (max(0, Ho - 7), max(0, Wo - 9)), (max(0, Ho // 2 - 3), max(0, Wo // 2 - 3)), (0, max(0, Wo - 9))}:
            yield n, h0, min(h0 + 7, Ho), w0, min(w0 + 9, Wo)


def conv_fused(layer, x, stride, coherent, scale, bias, res, out_dt, y, ld):
    if not coherent:
        return layer.conv_fused(x, stride=stride, scale=scale, bias=bias, act=B.ACT_SILU, residual=res, out_dt=out_dt, y=y)
    ep = B.EpilogueDesc(scale.data_ptr(), bias.data_ptr(), B.ACT_SILU, res.data_ptr(), ld, ld)
    c = B.CDesc(x.shape[0], x.shape[1], x.shape[2], stride, 1, B.NHWC, out_dt, 0)
    B.rtoss_conv2d_pattern_coherent(layer.wdesc, c, ep, layer.masks, layer.blob.data_ptr(), x.data_ptr(), y.data_ptr(),
                                    torch.cuda.current_stream().cuda_stream)


@pytest.mark.parametrize("case", VARIANTS, ids=lambda c: "%s-%s" % (c[0], wl.DTYPE_NAMES[c[1]]))
def test_variant(case):
    kernel, dt, N, Ci, Co, H, W, ks, stride, k, fused, coherent = case
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci + Co + H)
    rng = np.random.default_rng(Ci * 3 + Co + H)
    masks = B.rtoss_pattern_dict(k)
    T = pl.TORCH_DTYPE[dt]
    ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, ks, ks)) * (0.5 / np.sqrt(Ci)), dt)
    x = torch.randn((N, H, W, Ci), generator=g, device="cuda").to(T)
    if coherent:
        idx = np.repeat(rng.integers(0, len(masks), Ci // 8), 8)[None, :].repeat(Co, 0).astype(np.uint8).reshape(-1)
        layer = pl.CoherentLayer(Co, Ci, k, dt, masks).pack(pl.to_device(ws, dt), torch.from_numpy(idx).cuda())
        plain = layer
    else:
        own = GpuLayer(ws, dt, masks, k)
        idx, layer, plain = own.idx_host(), own.layer, own.layer
    pruned = oracle.mask(wl.to_f64(ws, dt), masks, idx)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1

    # the convolution alone
    y = plain.conv(x, stride=stride, relu=True, out_dt=wl.F32)
    if dt != wl.F32:
        assert torch.equal(plain.conv(x, stride=stride, relu=True), y.to(T))
    # with its output stage, between two runs of 8 channels of a wider buffer; the shortcut is exact in either type
    first, wide = 8, -(-Co // 8) * 8 + 16
    scale, bias = torch.rand(Co, generator=g, device="cuda") + 0.5, torch.randn(Co, generator=g, device="cuda")
    res = torch.randn((N, Ho, Wo, wide), generator=g, device="cuda").to(T)
    z = None
    if fused:
        z = torch.full((N, Ho, Wo, wide), 7.0, device="cuda")
        conv_fused(layer, x, stride, coherent, scale, bias, res.float()[..., first:first + Co], wl.F32, z[..., first:first + Co], wide)
        assert bool((z[..., :first] == 7.0).all()) and bool((z[..., first + Co:] == 7.0).all())
        if dt != wl.F32:
            z16 = torch.full((N, Ho, Wo, wide), 7.0, device="cuda", dtype=T)
            conv_fused(layer, x, stride, coherent, scale, bias, res[..., first:first + Co], dt, z16[..., first:first + Co], wide)
            assert torch.equal(z16, z.to(T))
    got, want, got_z, want_z = [], [], [], []
    for n, h0, h1, w0, w1 in windows(N, Ho, Wo):
        # input rows and columns with one output's worth of halo on the sides that have one, whose outputs are dropped
        top, left = int(h0 > 0), int(w0 > 0)
        rows, cols = slice((h0 - top) * stride, min(H, h1 * stride + 1)), slice((w0 - left) * stride, min(W, w1 * stride + 1))
        xin = wl.nhwc_to_nchw(x[n:n + 1, rows, cols].double().cpu().numpy())
        here = (slice(None), slice(None), slice(top, top + h1 - h0), slice(left, left + w1 - w0))
        want.append(oracle.conv2d(xin, pruned, stride=stride, relu=True)[here].ravel())
        got.append(wl.nhwc_to_nchw(y[n:n + 1, h0:h1, w0:w1].double().cpu().numpy()).ravel())
        if fused:
            ref = oracle.conv2d_fused(xin, pruned, stride=stride, scale=scale.cpu().numpy(), bias=bias.cpu().numpy(), act=B.ACT_SILU)[here]
            r = res[n:n + 1, h0:h1, w0:w1, first:first + Co].double().cpu().numpy()
            want_z.append((ref + wl.nhwc_to_nchw(r)).ravel())
            got_z.append(wl.nhwc_to_nchw(z[n:n + 1, h0:h1, w0:w1, first:first + Co].double().cpu().numpy()).ravel())
    check(np.concatenate(got), np.concatenate(want), dt)
    if fused:
        check(np.concatenate(got_z), np.concatenate(want_z), dt)
