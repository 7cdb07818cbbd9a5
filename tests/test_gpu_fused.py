"""GPU parity of the fused output stage: y = act(scale[co] * conv + bias[co]) + residual, for every
convolution kernel family, against the oracle's term-by-term definition."""
import zlib

import numpy as np
import pytest
import torch

import oracle
from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

from gpu_util import GpuLayer

pytestmark = pytest.mark.gpu

# kernel (test_routes.py checks it), dt, N, Ci, Co, H, W, ks, stride, k, rule: one case per kernel family and shape class
CASES = [
    ("conv3x3_rows", wl.BF16, 13, 128, 128, 52, 50, 3, 1, 3, B.RULE_CONNECTED4),  # (>= 200 tiles of 16x16 x 128 channels)
    ("conv3x3_rows", wl.F16, 7, 256, 272, 33, 49, 3, 1, 2, B.RULE_CONNECTED4),    # ragged tiles, padded channel block
    ("conv3x3_ksplit", wl.BF16, 1, 128, 128, 20, 24, 3, 1, 3, B.RULE_CONNECTED4),
    ("conv3x3_ksplit", wl.F16, 2, 64, 48, 19, 21, 3, 1, 3, B.RULE_CONNECTED4),
    ("conv3x3_ksplit", wl.BF16, 1, 128, 144, 37, 41, 3, 2, 2, B.RULE_CONNECTED4),  # stride 2
    ("conv3x3_ksplit", wl.F16, 1, 64, 80, 18, 20, 3, 1, 4, B.RULE_CONNECTED4),     # three tap groups
    ("conv3x3_ksplit", wl.BF16, 1, 96, 64, 21, 9, 3, 2, 5, B.RULE_CONNECTED4),     # one step per tap, stride 2
    ("conv3x3_sparse_sb", wl.F16, 17, 32, 16, 87, 83, 3, 1, 3, B.RULE_CONNECTED4),   # one buffer, one stage
    ("conv3x3_sparse_sb", wl.BF16, 17, 96, 16, 83, 87, 3, 1, 2, B.RULE_CONNECTED4),  # two buffers
    ("conv3x3_sparse_sb", wl.F16, 17, 32, 80, 19, 21, 3, 2, 3, B.RULE_CONNECTED4),   # stride 2
    ("conv3x3_sparse_sb", wl.BF16, 17, 64, 144, 21, 19, 3, 2, 4, B.RULE_CONNECTED4),  # ... three tap groups
    ("conv3x3_strip", wl.F16, 17, 64, 80, 19, 21, 3, 1, 3, B.RULE_CONNECTED4),
    ("conv3x3_dense", wl.BF16, 2, 32, 80, 18, 21, 3, 1, 5, B.RULE_CONNECTED4),
    ("conv3x3_dense", wl.F16, 17, 32, 80, 17, 19, 3, 2, 5, B.RULE_CONNECTED4),
    ("conv3x3_stem", wl.F16, 2, 3, 32, 33, 35, 3, 2, 2, B.RULE_CONNECTED4),
    ("conv1x1_stream", wl.F16, 3, 64, 32, 23, 17, 1, 1, 2, B.RULE_CONNECTED4),     # waves over positions
    ("conv1x1_stream", wl.BF16, 9, 256, 464, 13, 21, 1, 1, 2, B.RULE_CONNECTED4),  # ... over channels
    ("conv1x1_stream", wl.F16, 2, 512, 464, 23, 45, 1, 1, 3, B.RULE_CONNECTED4),   # two fragments per wave
    ("conv1x1_stream", wl.F16, 6, 1024, 400, 13, 17, 1, 1, 2, B.RULE_CONNECTED4),  # one fragment per wave, padded channels
    ("conv1x1_ksplit", wl.BF16, 2, 256, 256, 15, 13, 1, 1, 2, B.RULE_CONNECTED4),
    ("conv1x1_ksplit", wl.F16, 1, 512, 128, 11, 10, 1, 1, 3, B.RULE_CONNECTED4),
    ("conv1x1_ksplit", wl.F16, 1, 1024, 80, 7, 9, 1, 1, 2, B.RULE_CONNECTED4),
    ("conv1x1_mma", wl.BF16, 1, 96, 48, 13, 11, 1, 1, 2, B.RULE_CONNECTED4),
    ("conv3x3_dense", wl.F32, 1, 16, 24, 14, 15, 3, 1, 4, B.RULE_CONNECTED4),      # ragged channels out, fp32
    ("conv3x3_sparse_sb", wl.F16, 1, 24, 40, 9, 10, 3, 2, 3, B.RULE_CONNECTED4),   # ragged channels
    ("conv1x1_mma", wl.F32, 2, 40, 24, 8, 9, 1, 1, 2, B.RULE_CONNECTED4),          # ragged channels, fp32
    ("conv_direct", wl.F32, 1, 3, 16, 14, 15, 3, 1, 4, B.RULE_CONNECTED4),
]
STAGES = [
    dict(scale=True, bias=True, act=B.ACT_SILU, residual=True),
    dict(scale=False, bias=True, act=B.ACT_RELU, residual=False),
    dict(scale=True, bias=False, act=B.ACT_NONE, residual=False),
    dict(scale=False, bias=False, act=B.ACT_NONE, residual=True),
    dict(scale=False, bias=False, act=B.ACT_SILU, residual=False),
]


def _tolerance(ref, dt, out_dt):
    if dt == wl.F32:
        return 1e-5 * np.max(np.abs(ref))
    tol = 2e-3 * np.sqrt(np.mean(ref ** 2))
    if out_dt != wl.F32:  # one rounding of the stored value on top
        tol = tol + np.max(np.abs(ref)) * (2.0 ** -8 if out_dt == wl.BF16 else 2.0 ** -11)
    return tol


@pytest.mark.parametrize("stage", STAGES, ids=lambda s: "%s%s%d%s" % ("s" if s["scale"] else "-", "b" if s["bias"] else "-",
                                                                      s["act"], "r" if s["residual"] else "-"))
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s_dt%d_%dx%d_k%d_s%d_%d-%d" % (c[0], c[1], c[7], c[7], c[9], c[8], c[3], c[4]))
def test_fused_output_stage(case, stage):
    _, dt, N, Ci, Co, H, W, ks, stride, k, rule = case
    rng = np.random.default_rng(zlib.crc32(repr((case[1:], sorted(stage.items()))).encode()))  # the same inputs in every process
    masks = B.rtoss_pattern_dict(k, rule)
    xs = wl.round_to_dtype(rng.standard_normal((N, Ci, H, W)), dt)
    ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, ks, ks)) * (0.4 / np.sqrt(Ci)), dt)
    xv, wv = wl.to_f64(xs, dt), wl.to_f64(ws, dt)
    scale = rng.uniform(0.5, 1.5, Co).astype(np.float32) if stage["scale"] else None
    bias = rng.standard_normal(Co).astype(np.float32) if stage["bias"] else None
    g = GpuLayer(ws, dt, masks, k)
    pruned = oracle.mask(wv, masks, g.idx_host())
    x_dev = pl.to_device(wl.nchw_to_nhwc(xs), dt)
    sc_dev = torch.from_numpy(scale).cuda() if scale is not None else None
    bi_dev = torch.from_numpy(bias).cuda() if bias is not None else None
    for out_dt in ([wl.F32] if dt == wl.F32 else [wl.F32, dt]):
        ref0 = oracle.conv2d(xv, pruned, stride=stride)
        res_store = res_vals = res_dev = None
        if stage["residual"]:
            res_store = wl.round_to_dtype(rng.standard_normal(ref0.shape), out_dt)
            res_vals = wl.to_f64(res_store, out_dt)
            res_dev = pl.to_device(wl.nchw_to_nhwc(res_store), out_dt)
        ref = oracle.conv2d_fused(xv, pruned, stride=stride, scale=scale, bias=bias, act=stage["act"], residual=res_vals)
        y = g.layer.conv_fused(x_dev, stride=stride, scale=sc_dev, bias=bi_dev, act=stage["act"], residual=res_dev,
                               out_dt=out_dt)
        torch.cuda.synchronize()
        got = wl.to_f64(wl.nhwc_to_nchw(pl.to_host(y)), out_dt)
        assert got.shape == ref.shape
        err = np.max(np.abs(got - ref))
        assert err <= _tolerance(ref, dt, out_dt), (err, _tolerance(ref, dt, out_dt), out_dt)


def test_fused_relu_equals_the_plain_call_bit_for_bit():
    # act = ReLU through the fused entry point and fuse_relu through the plain one are the same arithmetic
    dt, k = wl.BF16, 3
    rng = np.random.default_rng(4)
    masks = B.rtoss_pattern_dict(k)
    for Ci, Co, ks, stride in [(128, 128, 3, 1), (64, 64, 3, 2), (256, 64, 1, 1)]:
        ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, ks, ks)) * 0.05, dt)
        xs = wl.round_to_dtype(rng.standard_normal((2, Ci, 18, 22)), dt)
        g = GpuLayer(ws, dt, masks, k)
        x_dev = pl.to_device(wl.nchw_to_nhwc(xs), dt)
        a = g.layer.conv(x_dev, stride=stride, relu=True)
        b = g.layer.conv_fused(x_dev, stride=stride, act=B.ACT_RELU)
        torch.cuda.synchronize()
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


# kernels, dt, N, Ci, Co_a, Co_b, H, W, ks, stride, k: two layers over one input write the two channel slices of one buffer
CONCAT_CASES = [
    ("conv3x3_rows+conv3x3_strip", wl.BF16, 13, 128, 128, 64, 52, 50, 3, 1, 3),
    ("conv3x3_ksplit+conv3x3_ksplit", wl.F16, 2, 64, 48, 16, 19, 21, 3, 1, 3),
    ("conv3x3_ksplit+conv3x3_ksplit", wl.BF16, 1, 128, 144, 32, 37, 41, 3, 2, 2),
    ("conv3x3_ksplit+conv3x3_ksplit", wl.F16, 1, 64, 80, 48, 18, 20, 3, 1, 4),
    ("conv3x3_sparse_sb+conv3x3_sparse_sb", wl.F16, 17, 32, 48, 16, 87, 83, 3, 1, 3),  # stride 1
    ("conv3x3_sparse_sb+conv3x3_sparse_sb", wl.BF16, 17, 32, 80, 144, 19, 21, 3, 2, 2),  # stride 2
    ("conv3x3_dense+conv3x3_dense", wl.F16, 2, 32, 80, 48, 18, 20, 3, 1, 5),
    ("conv3x3_stem+conv3x3_stem", wl.F16, 2, 3, 32, 16, 33, 35, 3, 2, 2),
    ("conv1x1_stream+conv1x1_stream", wl.F16, 3, 64, 32, 64, 23, 17, 1, 1, 2),
    ("conv1x1_stream+conv1x1_stream", wl.BF16, 9, 256, 464, 528, 13, 21, 1, 1, 2),  # waves over channels
    ("conv1x1_ksplit+conv1x1_ksplit", wl.BF16, 2, 256, 256, 128, 15, 13, 1, 1, 2),
    ("conv1x1_mma+conv1x1_mma", wl.BF16, 1, 96, 48, 16, 13, 11, 1, 1, 2),
    ("conv3x3_dense+conv3x3_dense", wl.F32, 1, 16, 24, 8, 14, 15, 3, 1, 4),  # ragged channels out, fp32
    ("conv3x3_sparse_sb+conv3x3_sparse_sb", wl.F16, 1, 24, 40, 8, 9, 10, 3, 2, 3),  # ragged channels
    ("conv_direct+conv_direct", wl.F32, 1, 3, 16, 8, 14, 15, 3, 1, 4),
]


@pytest.mark.parametrize("case", CONCAT_CASES, ids=lambda c: "%s_dt%d_s%d_%d-%d+%d" % (c[0], c[1], c[9], c[3], c[4], c[5]))
def test_two_layers_write_one_concatenation(case):
    """Section V.C times whole detectors, whose blocks concatenate branch outputs along channels: two
    convolutions write their channel slices of one channels-last buffer (y_ld = the buffer's channel count),
    the second adding a shortcut read from a slice of another wide buffer (residual_ld).  Both slices are
    compared with the oracle and the channels between and around them must keep their sentinel."""
    _, dt, N, Ci, Ca, Cb, H, W, ks, stride, k = case
    rng = np.random.default_rng(zlib.crc32(repr(case[1:]).encode()))
    masks = B.rtoss_pattern_dict(k)
    xs = wl.round_to_dtype(rng.standard_normal((N, Ci, H, W)), dt)
    xv = wl.to_f64(xs, dt)
    x_dev = pl.to_device(wl.nchw_to_nhwc(xs), dt)
    layers, pruned = [], []
    for Co in (Ca, Cb):
        ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, ks, ks)) * (0.4 / np.sqrt(Ci)), dt)
        g = GpuLayer(ws, dt, masks, k)
        layers.append(g)
        pruned.append(oracle.mask(wl.to_f64(ws, dt), masks, g.idx_host()))
    bias = rng.standard_normal(Cb).astype(np.float32)
    ref_a = oracle.conv2d_fused(xv, pruned[0], stride=stride, act=B.ACT_RELU)
    gap = 8  # untouched channels between the two slices
    for out_dt in ([wl.F32] if dt == wl.F32 else [wl.F32, dt]):
        tdt = pl.TORCH_DTYPE[out_dt]
        _, _, Ho, Wo = ref_a.shape
        res_store = wl.round_to_dtype(rng.standard_normal((N, Cb, Ho, Wo)), out_dt)
        res_wide = torch.full((N, Ho, Wo, Cb + 24), 7.0, dtype=tdt, device="cuda")
        res_wide[..., 16:16 + Cb] = pl.to_device(wl.nchw_to_nhwc(res_store), out_dt)
        ref_b = oracle.conv2d_fused(xv, pruned[1], stride=stride, bias=bias, act=B.ACT_SILU,
                                    residual=wl.to_f64(res_store, out_dt))
        total = Ca + gap + Cb + 8
        buf = torch.full((N, Ho, Wo, total), -3.0, dtype=tdt, device="cuda")
        ya, yb = buf[..., :Ca], buf[..., Ca + gap: Ca + gap + Cb]
        layers[0].layer.conv_fused(x_dev, stride=stride, act=B.ACT_RELU, out_dt=out_dt, y=ya)
        layers[1].layer.conv_fused(x_dev, stride=stride, bias=torch.from_numpy(bias).cuda(), act=B.ACT_SILU,
                                   residual=res_wide[..., 16:16 + Cb], out_dt=out_dt, y=yb)
        torch.cuda.synchronize()
        host = buf.cpu()
        assert bool((host[..., Ca:Ca + gap] == -3.0).all()) and bool((host[..., Ca + gap + Cb:] == -3.0).all())
        for ysl, ref in ((host[..., :Ca], ref_a), (host[..., Ca + gap: Ca + gap + Cb], ref_b)):
            got = wl.to_f64(wl.nhwc_to_nchw(pl.to_host(ysl.contiguous())), out_dt)
            err = np.max(np.abs(got - ref))
            assert err <= _tolerance(ref, dt, out_dt), (err, _tolerance(ref, dt, out_dt), out_dt)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s_dt%d_%dx%d_k%d_s%d_%d-%d" % (c[0], c[1], c[7], c[7], c[9], c[8], c[3], c[4]))
def test_silu_of_chosen_values(case):
    """With activations of zero the output stage's argument is the bias: SiLU over the whole range of fp32, where the
    correction of the reciprocal takes over from the division and beyond, and one rounding for 16-bit results."""
    _, dt, N, Ci, Co, H, W, ks, stride, k, rule = case
    rng = np.random.default_rng(Ci + Co)
    ends = np.array([0.0, 1e-45, -1e-45, 1e-38, -1e-38, 1e-30, 1.0, -1.0, 79.99999, 80.0, 80.00001, -79.99999, -80.0, -80.00001, -87.0,
                     -87.5, -88.5, -89.0, -104.0, -3e38, 3e38, np.inf, -np.inf, np.nan, 16.7, -16.7, 104.0, -60.0])
    bias = np.concatenate([ends, rng.standard_normal(Co) * 4])[rng.permutation(len(ends) + Co)][:Co].astype(np.float32)
    x = torch.zeros((N, H, W, Ci), dtype=pl.TORCH_DTYPE[dt], device="cuda")
    layer = GpuLayer(wl.round_to_dtype(rng.standard_normal((Co, Ci, ks, ks)), dt), dt, B.rtoss_pattern_dict(k, rule), k).layer
    b = torch.from_numpy(bias).cuda()
    y = layer.conv_fused(x, stride=stride, bias=b, act=B.ACT_SILU, out_dt=wl.F32)
    v = bias.astype(np.float64)
    with np.errstate(over="ignore", invalid="ignore"):
        want = v / (1.0 + np.exp(-v))
    got = y.cpu().numpy().astype(np.float64)
    # fp32 error of exp(-v): its argument's rounding (2^-24 of |v| / ln 2) and one unit; then an addition and a division.
    # Below -87 exp(-v) nears the end of the fp32 range and results are under 1e-36.
    bound = np.abs(want) * (np.abs(v) * 2.0 ** -23 + 2.0 ** -22) + 1e-36
    ok = (np.abs(got - want) <= bound) | (got == want) | (np.isnan(got) & np.isnan(want))
    assert ok.all(), (v[np.argwhere(~ok)[0][-1]], got[~ok][0])
    if dt != wl.F32:
        y16 = layer.conv_fused(x, stride=stride, bias=b, act=B.ACT_SILU)
        rounded = y.to(y16.dtype)
        assert bool(((y16 == rounded) | (y16.isnan() & rounded.isnan())).all())


@pytest.mark.parametrize("dt", [wl.F16, wl.BF16])
def test_16bit_silu_is_the_fp32_result_rounded_once(dt):
    """2.6 million outputs: a reciprocal in the place of the division would round a few dozen of them differently."""
    rng = np.random.default_rng(17)
    g = torch.Generator(device="cuda")
    g.manual_seed(17)
    layer = GpuLayer(wl.round_to_dtype(rng.standard_normal((64, 32, 1, 1)) * 0.4, dt), dt, B.rtoss_pattern_dict(3), 3).layer
    x = torch.randn((1, 200, 200, 32), generator=g, device="cuda").to(pl.TORCH_DTYPE[dt])
    bias = torch.randn(64, generator=g, device="cuda")
    y32 = layer.conv_fused(x, bias=bias, act=B.ACT_SILU, out_dt=wl.F32)
    y16 = layer.conv_fused(x, bias=bias, act=B.ACT_SILU)
    assert torch.equal(y16, y32.to(y16.dtype))
