"""The dispatch, replayed without a GPU: tests/variants.py names the kernel each of its calls launches, and together they
launch every convolution kernel the library holds, so that a change of a rule cannot empty a GPU test unnoticed."""
import pytest

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import workloads as wl

import routes
import test_gpu_both_sections
import test_gpu_conv
import test_gpu_fused
import test_gpu_ksplit
import test_gpu_ksplit1x1
import test_gpu_launch_limits
import test_gpu_rows_groups
import test_gpu_slices
import test_gpu_stream1x1
import test_gpu_stride2_rows
import test_gpu_strip
import test_gpu_strip_ring
from variants import OWN_TYPE_OUT, VARIANTS


def call(dt, N, Ci, Co, H, W, ks, stride, k, out_dt, fused, coherent=False, rule=B.RULE_CONNECTED4):
    return (dt, N, Ci, Co, H, W, ks, stride, k, rule, out_dt, int(fused), int(coherent))  # (fused: route_probe.cpp)


def split(kernel):
    """'conv3x3_strip<f16,f32,3,0,true>' -> ('conv3x3_strip<3,0,true>', 'f16')"""
    name, args = kernel[:-1].split("<")
    args = args.split(",")
    types = [a for a in args if a in ("f32", "f16", "bf16")]
    return "%s<%s>" % (name, ",".join(a for a in args if a not in types)), types[0]


def test_every_variant_is_reached_where_the_list_says():
    calls, want = [], []
    for kernel, dt, N, Ci, Co, H, W, ks, stride, k, fused, coherent in VARIANTS:
        for out_dt in ([dt] if kernel in OWN_TYPE_OUT or dt == wl.F32 else [wl.F32, dt]):
            calls.append(call(dt, N, Ci, Co, H, W, ks, stride, k, out_dt, fused, coherent))
            want.append((kernel, wl.DTYPE_NAMES[dt]))
    got = [split(k) for k in routes.kernels(calls)]
    assert [(c, g) for c, g, w in zip(calls, got, want) if g != w] == []


def test_the_list_covers_the_library():
    held = {(name, "f32" if dt == "f32" else "16-bit") for name, dt in map(split, routes.library_kernels("conv"))}
    listed = {(v[0], "f32" if v[1] == wl.F32 else "16-bit") for v in VARIANTS}
    held.discard(("conv_direct<1,1,0>", "f32"))  # NCHW tensors only
    assert held == listed


def test_launches_stay_within_the_lds_they_declare():
    """... and a compute unit has: every variant in both output types, and long output rows of 1x1 layers."""
    calls = [call(dt, N, Ci, Co, H, W, ks, stride, k, out_dt, fused, coherent)
             for kernel, dt, N, Ci, Co, H, W, ks, stride, k, fused, coherent in VARIANTS for out_dt in {wl.F32, dt}]
    for dt in (wl.F16, wl.BF16, wl.F32):
        for Ci in (18, 24):
            for Co in (129, 248, 255, 256, 517, 700, 2000, (1 << 24) + 8, (1 << 25) + 3):
                for H, W in ((1, 1), (131, 129)):
                    calls += [call(dt, 1, Ci, Co, H, W, 1, 1, 2, out_dt, fused) for out_dt in {wl.F32, dt} for fused in (False, True)]
    wrong = [(c, l) for c, l in zip(calls, routes.launches(calls)) if isinstance(l[0], str) and not l[1] <= l[2] <= 160 * 1024]
    assert wrong == []


def test_packing_allocates_nothing():
    """... so that no exception can leave the C interface there (the probe refuses every allocation and ends at the first)."""
    for dt in (wl.F32, wl.F16, wl.BF16):
        calls = [call(dt + 16, 1, Ci, 48, 9, 19, ks, 1, 3, dt, False) for Ci, ks in ((64, 3), (3, 3), (64, 1), (40, 1))]
        assert families(routes.kernels(calls)) == ["pack"] * len(calls)


def families(kernels):
    return [k if isinstance(k, int) else k.split("<")[0] for k in kernels]


@pytest.mark.parametrize("fused", [False, True])
def test_cases_made_for_a_kernel_reach_it(fused):
    for cases, kernel in ((test_gpu_strip.CASES, "conv3x3_strip"), (test_gpu_ksplit.CASES, "conv3x3_ksplit")):
        calls = [call(c[0], *c[1:6], 3, c[6] if len(c) == 8 else 1, c[-1], wl.F32, fused) for c in cases]
        assert families(routes.kernels(calls)) == [kernel] * len(cases)
    calls = [call(dt, N, Ci, Co, H, W, 1, 1, 2, wl.F32, fused) for dt, N, Ci, Co, H, W in test_gpu_ksplit1x1.CASES]
    assert families(routes.kernels(calls)) == ["conv1x1_ksplit"] * len(calls)
    calls = [call(c[0], *c[2:], 3, 2, c[1], c[0], fused) for c in test_gpu_stride2_rows.CASES]
    assert families(routes.kernels(calls)) == ["conv3x3_sparse_sb"] * len(calls)
    calls = [call(c[0], *c[2:], 3, 2, c[1], c[0], fused) for c in test_gpu_stride2_rows.RESIDENT_CASES]
    assert families(routes.kernels(calls)) == ["conv3x3_resident"] * len(calls)
    calls = [call(dt, 1, Ci, Co, 1, P, 1, 1, 2, out_dt, fused) for dt, Ci, Co, P in test_gpu_stream1x1.CASES for out_dt in (dt, wl.F32)]
    assert families(routes.kernels(calls)) == ["conv1x1_stream"] * len(calls)


def test_cases_reach_the_layout_they_name():
    """Rows and tap layout of the strips (2: dense mode, its weights in LDS; a number alone: past it, that many rows), steps of the channel split,
    blocks a wave and layout at stride 2."""
    def variants(calls):
        return [split(k)[0].split("<")[1][:-1].split(",") for k in routes.kernels(calls)]

    strips = ["2,0", "2,0", "3,0", "3,0", "4,0", "2,1", "3,1", "4,1", "5,1", "8", "2,1", "3,1", "4,1", "5,1", "2,2", "3,2", "4,2", "5,2", "8", "8"]
    for fused in (False, True):
        got = variants([call(c[0], *c[1:6], 3, 1, c[-1], wl.F32, fused) for c in test_gpu_strip.CASES])
        assert [",".join(v[:2]) for v in got] == strips
        got = variants([call(c[0], *c[1:6], 3, c[6], c[-1], wl.F32, fused) for c in test_gpu_ksplit.CASES])
        assert [v[-1] for v in got] == ["0"] * 10 + ["1"] * 8 + ["2"] * 7
        got = variants([call(c[0], *c[2:], 3, 2, c[1], c[0], fused) for c in test_gpu_stride2_rows.CASES])
        assert [(v[2], v[6]) for v in got] == [("1", "0")] * 3 + [("1", "1"), ("2", "0"), ("1", "1"), ("2", "1")]
        got = variants([call(*c[1:], c[1], fused) for c in test_gpu_slices.CASES if c[0] == "conv3x3_strip"])
        assert [v[0] if v[0] in ("16", "20") else v[1] for v in got] == ["1", "1", "1", "0", "1", "16", "20", "0"]
    dense_mode = [[split(k)[0] for k in routes.kernels([call(dt, *c[:5], 3, c[5], c[6], wl.F32, False, rule=c[7]) for c in test_gpu_conv.DENSE_MODE])]
                  for dt in (wl.F16, wl.BF16)]
    dense = "conv3x3_dense<1,1,1,4,false>"
    assert dense_mode[0] == dense_mode[1] == ["conv3x3_ksplit<1,1,1,2,1>"] * 2 + ["conv3x3_ksplit<1,2,1,2,1>", dense, dense, "conv3x3_ksplit<1,1,1,2,1>"] + \
        ["conv3x3_ksplit<2,2,1,1,1>"] * 2 + ["conv3x3_ksplit<2,2,1,1,2>", "conv3x3_ksplit<2,2,1,1,1>", dense]


RING_CASES = test_gpu_strip_ring.CASES + test_gpu_strip_ring.WIDE_CASES


def test_ring_cases_reach_the_height_they_name():
    calls = [call(dt, N, Ci, Co, H, W, 3, 1, k, dt, fused) for tn, dt, N, Ci, Co, H, W, k in RING_CASES for fused in (False, True)]
    want = ["conv3x3_ring<%d,%d>" % (c[0], c[-1] >= 4) for c in RING_CASES for fused in (False, True)]
    assert [split(k)[0] for k in routes.kernels(calls)] == want


def test_shallow_launches_of_two_rounds_stay_without_helpers():
    """Eight rows a workgroup go over the chip twice, 16 once: with helpers from five stages on, where they are as fast (four of 16: 3 % slower)."""
    for k, least in ((2, 5), (3, 5), (4, 5)):
        for stages in (3, 4, 5, 8):
            calls = [call(wl.BF16, N, 32 * stages, Co, H, W, 3, 1, k, wl.BF16, fused) for fused in (False, True)
                     for N, Co, H, W in ((1, 192, 100, 168), (4, 336, 40, 40), (2, 208, 80, 80), (17, 64, 43, 50))]
            want = "conv3x3_ring<4,%d>" % (k >= 4) if stages >= least else "conv3x3_strip<2,%d,true>" % (k >= 4)
            assert {split(r)[0] for r in routes.kernels(calls)} == {want}, (k, stages)


def test_streaming_cases_cover_the_turns():
    """The buffers of a workgroup in test_gpu_stream1x1's cases, with one helper wave and with two: one, two, three and more, with at
    least two and at most four workgroups a compute unit (16 positions a wave along positions; at least two buffers a workgroup)."""
    calls = [call(dt, 1, Ci, Co, 1, P, 1, 1, 2, dt, True) for dt, Ci, Co, P in test_gpu_stream1x1.CASES]
    turns = {1: set(), 2: set()}
    for (dt, Ci, Co, P), kernel in zip(test_gpu_stream1x1.CASES, routes.kernels(calls)):
        args = split(kernel)[0][:-1].split("<")[1].split(",")
        if len(args) == 1:
            continue  # (the fp32 kernel without helpers)
        KS, WM = int(args[0]), int(args[1])
        helpers = 2 if KS >= 8 or 4 // WM * KS >= 16 else 1
        buffers, blocks = -(-P * WM // 64), -(-Co // (16 * WM * {32: 1, 16: 2}.get(KS, 4)))
        for per_cu in (2, 3, 4):
            groups = max(1, min((buffers + 1) // 2, 256 * per_cu // blocks))
            turns[helpers] |= {min(4, buffers // groups), min(4, -(-buffers // groups))}
    assert turns == {1: {1, 2, 3, 4}, 2: {1, 2, 3, 4}}


def test_slices_reach_the_kernel_they_name():
    for kernel, dt, N, Ci, Co, H, W, ks, stride, k in test_gpu_slices.CASES:
        for out_dt in {wl.F32, dt}:
            for fused in (False, True):
                assert families(routes.kernels([call(dt, N, Ci, Co, H, W, ks, stride, k, out_dt, fused)])) == [kernel]


def test_fused_cases_reach_the_kernel_they_name():
    for kernel, dt, N, Ci, Co, H, W, ks, stride, k, rule in test_gpu_fused.CASES:
        for out_dt in {wl.F32, dt}:
            assert families(routes.kernels([call(dt, N, Ci, Co, H, W, ks, stride, k, out_dt, True, rule=rule)])) == [kernel]
    for kernels, dt, N, Ci, Ca, Cb, H, W, ks, stride, k in test_gpu_fused.CONCAT_CASES:
        for out_dt in {wl.F32, dt}:
            got = routes.kernels([call(dt, N, Ci, Co, H, W, ks, stride, k, out_dt, True) for Co in (Ca, Cb)])
            assert families(got) == kernels.split("+")


def test_calls_past_launch_limits_leave_the_kernel_with_the_limit():
    calls = [call(dt, N, Ci, Co, H, W, ks, stride, k, dt, False) for dt, N, H, W, Ci, Co, ks, stride, k in test_gpu_launch_limits.CASES]
    assert families(routes.kernels(calls)) == ["conv_direct"] * 4 + ["conv1x1_stream", "conv3x3_dense"]
    # one row, column or image less, where that is below the limit
    below = [(wl.F16, 1, 46330, 46330, 8, 4, 3, 2, 3), (wl.BF16, 65280, 1, 4112, 8, 8, 3, 1, 2), (wl.F32, 1, (1 << 26) - 64, 1, 4, 4, 3, 1, 3),
             (wl.F16, 64800, 182, 182, 2, 1, 1, 1, 2)]
    calls = [call(dt, N, Ci, Co, H, W, ks, stride, k, dt, False) for dt, N, H, W, Ci, Co, ks, stride, k in below]
    assert families(routes.kernels(calls)) == ["conv3x3_sparse_sb", "conv3x3_sparse_sb", "conv3x3_dense", "conv1x1_mma"]


def test_cases_of_three_groups_reach_the_pipelined_kernel():
    calls = [call(dt, N, Ci, Co, H, W, 3, 1, k, out_dt, fused) for dt, N, Ci, Co, H, W, k in test_gpu_rows_groups.CASES
             for out_dt in (dt, wl.F32) for fused in (False, True)]
    assert families(routes.kernels(calls)) == ["conv3x3_rows"] * len(calls)
    # launches whose tiles would be mostly empty stay with the strips
    calls = [call(wl.BF16, N, Ci, Co, H, W, 3, 1, 4, wl.BF16, False) for N, Ci, Co, H, W in
             ((200, 96, 112, 5, 3), (200, 128, 128, 8, 16), (40, 96, 256, 24, 17), (4, 160, 144, 112, 162), (2, 128, 256, 33, 330))]
    assert families(routes.kernels(calls)) == ["conv3x3_strip"] * len(calls)


def test_layers_with_both_sections_take_the_faster_one():
    """Dictionaries that need repeated taps: by the shape alone, so that results of either type, with an output stage or into a slice, add in
    one order.  Dense mode: conv3x3_dense, layout 2 of the K split and of the strips, strips named by their rows."""
    def mode(kernel):
        name, args = split(kernel)[0][:-1].split("<")
        args = [a for a in args.split(",") if a not in ("true", "false")]
        if name in ("conv3x3_sparse_sb", "conv3x3_rows", "conv3x3_ksplit"):
            return "dense" if args[-1] == "2" else "2-of-4"
        return "dense" if name == "conv3x3_dense" or len(args) == 1 or args[1] == "2" else "2-of-4"

    for want, stride, shapes in test_gpu_both_sections.ROUTES:
        for N, Ci, Co, H, W in shapes:
            calls = [call(dt, N, Ci, Co, H, W, 3, stride, 5, out_dt, fused) for dt in (wl.F16, wl.BF16) for out_dt in (dt, wl.F32)
                     for fused in (0, 1, -(1 << 25))]
            assert {mode(k) for k in routes.kernels(calls)} == {want}, (N, Ci, Co, H, W, stride)
    # past the 2-of-4 kernels' limits (chunks of input; workgroups): the dense kernel
    calls = [call(wl.BF16, N, 64, 128, H, W, 3, stride, 5, wl.BF16, False)
             for N, H, W, stride in ((1, 16385, 16400, 1), (65535, 66, 64, 2), (65535, 1, 2064, 1))]
    assert families(routes.kernels(calls)) == ["conv3x3_dense"] * len(calls)


def test_wide_tile_reaches_the_pipelined_kernel():
    s = test_gpu_launch_limits.WIDE_TILE
    calls = [call(wl.F16, s["N"], s["Ci"], s["Co"], s["H"], s["W"], s["ks"], s["stride"], s["k"], out_dt, fused)
             for out_dt, fused in ((wl.F16, True), (wl.F32, True), (wl.F32, False))]
    assert families(routes.kernels(calls)) == ["conv3x3_rows"] * 3


def test_output_pitches_past_32_bit_offsets():
    """Kernels that store whole rows at 32-bit offsets take a call up to the longest pitch of which 64 positions are within them, and
    no further; those that do not are not asked to leave it.  (A pitch: more than 1 with a whole output stage, less than 0 alone.)"""
    for case in test_gpu_launch_limits.PITCH_CASES:
        dt, out_dt, N, Ci, Co, H, W, ks, stride, k, fused, coherent, within, beyond = case
        longest = (0xffffff00 - 1) // 64 // 64 * 64 // wl.ELEM_BYTES[out_dt]  # (whole sectors of 64 bytes)
        for pitch, want in ((longest, within), (longest + 64, beyond)):
            got = routes.kernels([call(dt, N, Ci, Co, H, W, ks, stride, k, out_dt, pitch if fused else -pitch, coherent)])[0]
            assert split(got)[0] == want, (case, pitch)
    # larger launches than a test has memory for; the resident stride-2 kernel's own limit: four rows of outputs
    for call_args, longest, within, beyond in (
            ((wl.F32, 1, 64, 64, 160, 160, 1, 1, 2, wl.F32), (0xffffff00 - 1) // 256 // 16 * 16, "conv1x1_stream<4>", "conv_direct<1,1,0>"),
            ((wl.BF16, 1, 512, 16, 120, 130, 1, 1, 2, wl.F32), (0xffffff00 - 1) // 256 // 16 * 16, "conv1x1_stream<16,2>", "conv1x1_stream<16,2>"),
            ((wl.BF16, 1, 512, 16, 120, 130, 1, 1, 2, wl.BF16), (0xffffff00 - 1) // 128 // 32 * 32, "conv1x1_stream<16,2>", "conv_direct<1,1,0>"),
            ((wl.F16, 1, 64, 448, 180, 180, 3, 2, 2, wl.F16), (0xffffff00 - 1) // (2 * (3 * 90 + 4)) // 32 * 32, "conv3x3_resident<2>",
             "conv3x3_sparse_sb<2,4,1,1,4,true,0,false,false>")):
        got = routes.kernels([call(*call_args, -pitch) for pitch in (longest, longest + 64)])
        assert [split(g)[0] for g in got] == [within, beyond]
