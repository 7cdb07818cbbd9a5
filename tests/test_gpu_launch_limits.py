"""Calls past the launch limits of a matrix-core kernel that took its shapes over from a kernel without them: more 16-byte
chunks than a 32-bit offset numbers, more workgroups than a grid holds.  They go where they went before."""
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
    # dt, N, H, W, Ci, Co, ks, stride, k
    (wl.F16, 1, 46344, 46344, 8, 4, 3, 2, 3),       # ragged 3x3: 2^31 chunks of input
    (wl.BF16, 65535, 1, 4112, 8, 8, 3, 1, 2),       # ... 2^24 workgroups
    (wl.F32, 1, (1 << 26) + 64, 1, 4, 4, 3, 1, 3),  # ragged 3x3, dense mode: 2^24 workgroups
    (wl.F16, 65535, 182, 182, 2, 1, 1, 1, 2),       # ragged 1x1: 2^24 workgroups
    (wl.F32, 1, 2800, 3000, 64, 1024, 1, 1, 2),     # fp32 1x1: 2^24 workgroups with the input channels split over waves
    (wl.BF16, 65535, 1, 4112, 64, 16, 3, 1, 5),     # strips of rows, dense mode: both
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "dt%d_%dx%dx%d_%d-%d_%dx%d" % (c[:6] + (c[6], c[6])))
def test_calls_past_a_kernels_launch_limits(case):
    dt, N, H, W, Ci, Co, ks, stride, k = case
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    torch.cuda.empty_cache()
    need = (N * H * W * Ci + N * Ho * Wo * Co) * wl.ELEM_BYTES[dt]
    if torch.cuda.mem_get_info()[0] < need + (4 << 30):
        pytest.skip("needs %d GB of device memory" % (need >> 30))
    rng = np.random.default_rng(N + H)
    masks = B.rtoss_pattern_dict(k)
    ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, ks, ks)), dt)
    layer = GpuLayer(ws, dt, masks, k)
    pruned = oracle.mask(wl.to_f64(ws, dt), masks, layer.idx_host())
    # zeros with a few islands: the first and last positions, and one in the middle (at even rows and columns)
    x = torch.zeros((N, H, W, Ci), dtype=pl.TORCH_DTYPE[dt], device="cuda")
    islands = []
    for n, h, w in ((0, 0, 0), (N // 2, H // 4 * 2, W // 4 * 2), (N - 1, max(0, H - 6) // 2 * 2, max(0, W - 8) // 2 * 2)):
        v = wl.round_to_dtype(rng.standard_normal((1, Ci, min(6, H - h), min(8, W - w))), dt)
        x[n:n + 1, h:h + v.shape[2], w:w + v.shape[3]] = pl.to_device(wl.nchw_to_nhwc(v), dt)
        islands.append((n, h, w, wl.to_f64(v, dt)))
    y = layer.layer.conv(x, stride=stride)
    nonzero = 0
    for n, h, w, v in islands:
        pad = [(0, 0), (0, 0), (2 * (h > 0), 2 * (h + v.shape[2] < H)), (2 * (w > 0), 2 * (w + v.shape[3] < W))]
        ref = oracle.conv2d(np.pad(v, pad), pruned, stride=stride)  # with the zeros around it, as far as they are in the image
        h0, w0 = (h - pad[2][0]) // stride, (w - pad[3][0]) // stride
        got = wl.nhwc_to_nchw(pl.to_host(y[n:n + 1, h0:h0 + ref.shape[2], w0:w0 + ref.shape[3]]))
        assert got.shape == ref.shape
        # fp32 accumulation of at most 9 * Ci products, then the rounding of the stored value
        bound = 1e-5 * np.max(np.abs(ref)) + np.abs(ref) * {wl.F32: 0.0, wl.F16: 2.0 ** -11, wl.BF16: 2.0 ** -8}[dt]
        assert (np.abs(wl.to_f64(got, dt) - ref) <= bound).all()
        nonzero += np.count_nonzero(got)
    assert sum(int(torch.count_nonzero(part)) for part in y.flatten().split(1 << 30)) == nonzero
    del x, y
    torch.cuda.empty_cache()


# Output pitches past the 32-bit offsets of stores in whole rows: dt, out_dt, N, Ci, Co, H, W, ks, stride, k, fused, coherent; the kernel
# while 64 positions are within 32 bits, and beyond (test_routes.py)
PITCH_CASES = [
    (wl.F16, wl.F16, 1, 64, 48, 1, 70, 1, 1, 2, True, False, "conv1x1_stream<2,1,false>", "conv1x1_stream<2,1,false>"),
    (wl.F16, wl.F16, 1, 128, 640, 4, 500, 1, 1, 2, True, False, "conv1x1_stream<4,4>", "conv_direct<1,1,0>"),
    (wl.F32, wl.F32, 1, 16, 64, 1, 70, 1, 1, 2, True, False, "conv1x1_stream<1,1>", "conv1x1_stream<1,1,false>"),
    (wl.F16, wl.F16, 1, 72, 32, 1, 70, 1, 1, 2, False, False, "conv1x1_mma<1,2,true>", "conv1x1_mma<1,2,true>"),
    (wl.F16, wl.F16, 1, 128, 16512, 20, 16, 3, 1, 3, False, False, "conv3x3_rows<false,0>", "conv3x3_sparse_sb<1,4,2,2,4,true,0,true,false>"),
    (wl.F16, wl.F16, 1, 128, 16512, 20, 16, 3, 1, 3, True, False, "conv3x3_rows<true,0>", "conv3x3_rows<true,0>"),
    (wl.BF16, wl.BF16, 1, 128, 8192, 20, 16, 3, 1, 3, True, False, "conv3x3_ring<3,0>", "conv3x3_sparse_sb<1,4,2,2,4,true,0,true,false>"),
    (wl.BF16, wl.BF16, 1, 128, 16384, 20, 16, 3, 1, 6, False, False, "conv3x3_strip<20,true>", "conv3x3_strip<20>"),
    (wl.F16, wl.F16, 1, 128, 16512, 20, 16, 3, 1, 5, False, False, "conv3x3_rows<false,1>", "conv3x3_strip<5,1,false>"),
    (wl.F32, wl.F32, 1, 64, 16384, 20, 16, 3, 1, 3, False, False, "conv3x3_strip<8>", "conv3x3_dense<1,1,1,4,false>"),
    (wl.F32, wl.F32, 1, 64, 2048, 20, 16, 3, 1, 3, True, False, "conv3x3_dense<1,4,false>", "conv3x3_dense<1,1,1,4,false>"),
    (wl.BF16, wl.BF16, 1, 256, 16384, 20, 16, 3, 1, 3, False, True, "conv3x3_gather_rows<>", "conv3x3_gather<1>"),
    (wl.BF16, wl.BF16, 1, 128, 32, 1, 70, 3, 1, 2, True, False, "conv3x3_ksplit<1,1,1,2,0>", "conv3x3_ksplit<1,1,1,2,0>"),
    (wl.F16, wl.F16, 1, 3, 32, 9, 17, 3, 1, 2, True, False, "conv3x3_stem<1,2,3>", "conv3x3_stem<1,2,3>"),
]


@pytest.mark.parametrize("case", PITCH_CASES, ids=lambda c: "-".join(map(str, c[:10])))
@pytest.mark.parametrize("rows", [64, 15], ids=lambda r: "%d_rows" % r)
def test_output_pitch_past_32_bit_offsets(case, rows):
    """Positions so far apart that 64 (15) of them span 4 GiB, where an offset of 32 bits would wrap: equal within the rounding of the
    stored value and the fp32 sums (another kernel may take the call)."""
    dt, out_dt, N, Ci, Co, H, W, ks, stride, k, fused, coherent = case[:12]
    P, eb = H * W, wl.ELEM_BYTES[out_dt]
    pitch = -(-(1 << 32) // rows // (eb * 16)) * 16
    if rows == 15 and P > 400:
        pytest.skip("64 rows apart are enough for a buffer of %d GB" % (P * pitch * eb >> 30))
    torch.cuda.empty_cache()
    if P * pitch * eb + (4 << 30) > torch.cuda.mem_get_info()[0]:
        pytest.skip("needs %d GB of device memory" % (P * pitch * eb >> 30))
    rng = np.random.default_rng(Ci)
    masks = B.rtoss_pattern_dict(k)
    ws = wl.round_to_dtype(rng.standard_normal((Co, Ci, ks, ks)) / np.sqrt(Ci * k), dt)
    packed = GpuLayer(ws, dt, masks, k)
    layer = packed.layer
    x = pl.to_device(wl.round_to_dtype(rng.standard_normal((N, H, W, Ci)), dt), dt)
    stage = dict(scale=torch.rand(Co, device="cuda") + 0.5, bias=torch.randn(Co, device="cuda"), act=B.ACT_SILU) if fused else {}
    wide = torch.empty((N, H, W, pitch), dtype=pl.TORCH_DTYPE[out_dt], device="cuda")
    wide[..., Co:Co + 64] = 7
    near = layer.conv_fused(x, out_dt=out_dt, **stage).float()
    if coherent:
        layer = pl.CoherentLayer(Co, Ci, k, dt, masks).pack(packed.w, packed.idx)
        e = B.EpilogueDesc(None, None, B.ACT_NONE, None, pitch, 0)
        B.rtoss_conv2d_pattern_coherent(layer.wdesc, B.CDesc(N, H, W, stride, ks // 2, B.NHWC, out_dt, 0), e, masks, layer.blob.data_ptr(),
                                        x.data_ptr(), wide.data_ptr(), torch.cuda.current_stream().cuda_stream)
        got = wide[..., :Co].float()
    else:
        got = layer.conv_fused(x, out_dt=out_dt, y=wide[..., :Co], **stage).float()
    peak = float(near.abs().max())
    bound = 1e-5 * peak + near.abs() * {wl.F32: 0.0, wl.F16: 2.0 ** -10, wl.BF16: 2.0 ** -7}[out_dt]
    assert ((got - near).abs() <= bound).all()
    assert (wide[..., Co:Co + 64] == 7).all()
    del wide
    torch.cuda.empty_cache()


# The pipelined 3x3 kernel's output through LDS (a fused stage, fp32 results): a tile of 20 rows of 16 positions.
WIDE_TILE = dict(N=1, H=20, W=16, Ci=128, Co=16512, ks=3, stride=1, k=3)


@pytest.mark.parametrize("out_dt,fused", [(wl.F16, True), (wl.F32, True), (wl.F32, False)])
def test_output_pitch_past_31_bit_elements(out_dt, fused):
    """Positions so far apart that those of one tile pass 2^31 elements: the same bits as side by side."""
    s = WIDE_TILE
    P, Co = s["H"] * s["W"], s["Co"]
    pitch = (1 << 31) // (P - 20) // 8 * 8  # the tile's last 20 positions lie beyond
    assert (P - 1) * pitch >= 1 << 31
    torch.cuda.empty_cache()
    need = P * pitch * wl.ELEM_BYTES[out_dt]
    if torch.cuda.mem_get_info()[0] < need + (2 << 30):
        pytest.skip("needs %d GB of device memory" % (need >> 30))
    rng = np.random.default_rng(P)
    masks = B.rtoss_pattern_dict(s["k"])
    layer = GpuLayer(wl.round_to_dtype(rng.standard_normal((Co, s["Ci"], 3, 3)) / 16, wl.F16), wl.F16, masks, s["k"]).layer
    x = pl.to_device(wl.round_to_dtype(rng.standard_normal((1, s["H"], s["W"], s["Ci"])), wl.F16), wl.F16)
    stage = {}
    if fused:
        stage = dict(scale=torch.rand(Co, device="cuda") + 0.5, bias=torch.randn(Co, device="cuda"), act=B.ACT_SILU)
    wide = torch.empty((1, s["H"], s["W"], pitch), dtype=pl.TORCH_DTYPE[out_dt], device="cuda")
    wide[..., Co:Co + 64] = 7
    got = layer.conv_fused(x, out_dt=out_dt, y=wide[..., :Co], **stage)
    assert torch.equal(got, layer.conv_fused(x, out_dt=out_dt, **stage))
    assert (wide[..., Co:Co + 64] == 7).all()
    del wide, got
    torch.cuda.empty_cache()
