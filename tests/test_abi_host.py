"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol
the header declares, generates the same dictionary as the oracle, and rejects bad arguments
before touching the GPU."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

import oracle
from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "rtoss.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(rtoss_[a-z0-9_]+)\s*\(", hdr))
    assert {"rtoss_select_patterns", "rtoss_pack", "rtoss_conv2d_pattern"} <= declared
    L = B.lib()
    for name in declared:
        assert hasattr(L, name), name
    assert declared == set(B.EXPORTS)


@pytest.mark.parametrize("rule", [0, 1, 2, 3])
@pytest.mark.parametrize("k", range(1, 10))
def test_dictionary_matches_oracle(k, rule):
    assert B.rtoss_pattern_dict(k, rule).tolist() == oracle.pattern_dict(k, rule).tolist()


def test_dictionary_errors():
    P = ctypes.c_int(0)
    L = B.lib()
    assert L.rtoss_pattern_dict(0, 2, None, 0, ctypes.byref(P)) == B.EINVAL
    assert L.rtoss_pattern_dict(3, 9, None, 0, ctypes.byref(P)) == B.EINVAL
    assert L.rtoss_pattern_dict(3, 2, None, 0, None) == B.EINVAL
    assert L.rtoss_pattern_dict(3, 2, None, 4, ctypes.byref(P)) == B.EINVAL
    buf = (ctypes.c_uint16 * 4)()
    assert L.rtoss_pattern_dict(3, 2, buf, 4, ctypes.byref(P)) == B.ENOSPACE
    assert P.value == 22 and list(buf) == oracle.pattern_dict(3).tolist()[:4]
    assert "22" in B.rtoss_last_error()


def _status(fn, *a, **kw):
    try:
        fn(*a, **kw)
    except B.RtossError as e:
        return e.status
    return B.OK


def test_select_argument_errors():
    masks = B.rtoss_pattern_dict(3)
    fake = 0x1000  # never dereferenced: every case below fails validation first
    assert _status(B.rtoss_select_patterns, fake, 7, 90, masks, fake) == B.EDTYPE
    assert _status(B.rtoss_select_patterns, fake, B.F16, -1, masks, fake) == B.EINVAL
    assert _status(B.rtoss_select_patterns, fake, B.F16, 90, None, fake) == B.EINVAL
    assert _status(B.rtoss_select_patterns, fake, B.F16, 90, np.zeros(0, np.uint16), fake) == B.EINVAL
    assert _status(B.rtoss_select_patterns, fake, B.F16, 90, np.ones(256, np.uint16), fake) == B.EINVAL
    assert _status(B.rtoss_select_patterns, fake, B.F16, 90, np.array([7, 3], np.uint16), fake) == B.EINVAL  # mixed k
    assert _status(B.rtoss_select_patterns, fake, B.F16, 90, np.array([0x200], np.uint16), fake) == B.EINVAL
    assert _status(B.rtoss_select_patterns, fake, B.F16, 90, np.array([0], np.uint16), fake) == B.EINVAL
    assert _status(B.rtoss_select_patterns, 0, B.F16, 90, masks, fake) == B.EINVAL
    assert _status(B.rtoss_select_patterns, fake, B.F16, 90, masks, 0) == B.EINVAL
    assert _status(B.rtoss_select_patterns, fake + 1, B.F16, 90, masks, fake) == B.EINVAL  # misaligned
    # fewer than 9 elements: nothing to do, pointers are not looked at
    assert _status(B.rtoss_select_patterns, 0, B.F16, 8, masks, 0) == B.OK


def test_pack_size_and_pack_errors():
    masks = B.rtoss_pattern_dict(3)
    d = B.WDesc(64, 32, 3, 3, B.F16)
    nbytes, ws = B.rtoss_pack_size(d, masks)
    assert nbytes >= 64 * 32 * (3 * 2 + 1) and nbytes % 256 == 0
    assert _status(B.rtoss_pack_size, B.WDesc(64, 32, 5, 3, B.F16), masks) == B.ESHAPE
    assert _status(B.rtoss_pack_size, B.WDesc(0, 32, 3, 3, B.F16), masks) == B.ESHAPE
    assert _status(B.rtoss_pack_size, B.WDesc(64, 32, 3, 2, B.F16), masks) == B.EINVAL  # k != popcount
    assert _status(B.rtoss_pack_size, B.WDesc(64, 32, 3, 3, 9), masks) == B.EDTYPE
    assert _status(B.rtoss_pack_size, None, masks) == B.EINVAL
    fake = 0x10000
    assert _status(B.rtoss_pack, d, fake, fake, masks, fake, nbytes - 1) == B.ENOSPACE
    assert _status(B.rtoss_pack, d, fake, fake, masks, 0, nbytes) == B.EINVAL
    assert _status(B.rtoss_pack, d, fake, fake, masks, fake + 16, nbytes) == B.EINVAL  # blob alignment
    assert _status(B.rtoss_pack, d, 0, fake, masks, fake, nbytes) == B.EINVAL
    assert _status(B.rtoss_pack, d, fake, 0, masks, fake, nbytes) == B.EINVAL


def test_conv_argument_errors():
    masks = B.rtoss_pattern_dict(3)
    d = B.WDesc(64, 32, 3, 3, B.F16)
    fake_p, fake_x, fake_y = 0x10000, 0x200000, 0x4000000
    good = dict(N=1, H=16, W=16, stride=1, pad=1, layout=B.NHWC, out_dt=B.F16, fuse_relu=0)

    def cd(**kw):
        a = dict(good)
        a.update(kw)
        return B.CDesc(a["N"], a["H"], a["W"], a["stride"], a["pad"], a["layout"], a["out_dt"], a["fuse_relu"])

    call = B.rtoss_conv2d_pattern
    assert _status(call, d, cd(layout=7), masks, fake_p, fake_x, fake_y) == B.EINVAL  # unknown layout
    assert _status(call, d, cd(stride=3), masks, fake_p, fake_x, fake_y) == B.ESHAPE
    assert _status(call, d, cd(pad=0), masks, fake_p, fake_x, fake_y) == B.ESHAPE
    assert _status(call, d, cd(N=0), masks, fake_p, fake_x, fake_y) == B.ESHAPE
    assert _status(call, d, cd(out_dt=B.BF16), masks, fake_p, fake_x, fake_y) == B.EDTYPE
    assert _status(call, d, None, masks, fake_p, fake_x, fake_y) == B.EINVAL
    assert _status(call, d, cd(), masks, 0, fake_x, fake_y) == B.EINVAL
    assert _status(call, d, cd(), masks, fake_p, fake_x + 2, fake_y) == B.EINVAL
    assert _status(call, d, cd(), masks, fake_p, fake_x, fake_x + 64) == B.EINVAL  # overlap
    assert _status(call, d, cd(), B.rtoss_pattern_dict(2), fake_p, fake_x, fake_y) == B.EINVAL  # k mismatch
    d1 = B.WDesc(64, 32, 1, 3, B.F16)
    assert _status(call, d1, cd(stride=2, pad=0), masks, fake_p, fake_x, fake_y) == B.ESHAPE


def test_reduce_dict_matches_oracle_and_rejects_bad_arguments():
    # host-only entry point: ranking by count, ties to the lower index, original order kept
    rng = np.random.default_rng(5)
    for k in (2, 3, 4):
        masks = B.rtoss_pattern_dict(k)
        for trial in range(5):
            counts = rng.integers(0, 6, len(masks)).astype(np.uint32)  # small range: many ties
            for M in (1, 2, len(masks) // 2, len(masks)):
                out, kept = B.rtoss_reduce_dict(masks, counts, M)
                want, want_kept = oracle.reduce_dict(masks, counts, M)
                assert out.tolist() == want.tolist() and kept.tolist() == want_kept.tolist()
    masks = B.rtoss_pattern_dict(2)
    counts = np.zeros(len(masks), dtype=np.uint32)
    for bad_M in (0, -1, len(masks) + 1):
        with pytest.raises(B.RtossError) as e:
            B.rtoss_reduce_dict(masks, counts, bad_M)
        assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError):
        B.rtoss_reduce_dict(masks, None, 3)
    with pytest.raises(B.RtossError):
        B.rtoss_reduce_dict(None, counts, 3)


def test_histogram_argument_errors():
    # validated on the host before any GPU call
    for args in [(0, 10, 12, 0), (256, -1, 12, 256), (256, 10, 0, 256), (256, 10, 256, 256), (256, 10, 12, 258)]:
        with pytest.raises(B.RtossError) as e:
            B.rtoss_pattern_histogram(*args)
        assert e.value.status == B.EINVAL
    B.rtoss_pattern_histogram(0, 0, 12, 256)  # nothing to count: no launch, no error


def test_batched_select_argument_errors():
    masks = B.rtoss_pattern_dict(2)
    with pytest.raises(B.RtossError) as e:
        B.rtoss_select_patterns_batch(None, B.F16, masks)  # NULL table with a non-zero count
    assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError) as e:
        B.rtoss_select_patterns_batch([(0, 900, 256)], B.F16, masks)  # NULL weights
    assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError) as e:
        B.rtoss_select_patterns_batch([(257, 900, 256)], B.F16, masks)  # misaligned weights
    assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError) as e:
        B.rtoss_select_patterns_batch([(256, -9, 256)], B.F16, masks)
    assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError) as e:
        B.rtoss_select_patterns_batch([(256, 900, 256)], 7, masks)
    assert e.value.status == B.EDTYPE
    B.rtoss_select_patterns_batch([], B.F16, masks)             # nothing to do
    B.rtoss_select_patterns_batch([(0, 8, 0)], B.F16, masks)    # fewer than 9 weights: no group, no launch


def test_fused_conv_argument_errors():
    masks = B.rtoss_pattern_dict(2)
    wd = B.WDesc(32, 32, 3, 2, B.F16)
    ok = B.CDesc(1, 8, 8, 1, 1, B.NHWC, B.F16, 0)
    good = B.EpilogueDesc(None, None, B.ACT_SILU, None)
    with pytest.raises(B.RtossError) as e:
        B.rtoss_conv2d_pattern_fused(wd, ok, None, masks, 256, 512, 1024)
    assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError) as e:  # fuse_relu together with an epilogue
        B.rtoss_conv2d_pattern_fused(wd, B.CDesc(1, 8, 8, 1, 1, B.NHWC, B.F16, 1), good, masks, 256, 512, 1 << 20)
    assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError) as e:  # unknown activation
        B.rtoss_conv2d_pattern_fused(wd, ok, B.EpilogueDesc(None, None, 9, None), masks, 256, 512, 1 << 20)
    assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError) as e:  # misaligned scale
        B.rtoss_conv2d_pattern_fused(wd, ok, B.EpilogueDesc(4, None, 0, None), masks, 256, 512, 1 << 20)
    assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError) as e:  # residual overlapping the output
        B.rtoss_conv2d_pattern_fused(wd, ok, B.EpilogueDesc(None, None, 0, (1 << 20) + 64), masks, 256, 512, 1 << 20)
    assert e.value.status == B.EINVAL
    # output / residual pitches (channel slices of wider buffers)
    for ep, want in [(B.EpilogueDesc(None, None, 0, None, 16, 0), B.ESHAPE),      # below Co
                     (B.EpilogueDesc(None, None, 0, None, 0, 24), B.ESHAPE),
                     (B.EpilogueDesc(None, None, 0, None, 36, 0), B.EINVAL),      # not a multiple of 16 bytes
                     (B.EpilogueDesc(None, None, 0, None, -8, 0), B.EINVAL)]:
        with pytest.raises(B.RtossError) as e:
            B.rtoss_conv2d_pattern_fused(wd, ok, ep, masks, 256, 512, 1 << 20)
        assert e.value.status == want
    with pytest.raises(B.RtossError) as e:  # pitches describe channels-last tensors
        B.rtoss_conv2d_pattern_fused(wd, B.CDesc(1, 8, 8, 1, 1, B.NCHW, B.F16, 0), B.EpilogueDesc(None, None, 0, None, 64, 0),
                                     masks, 256, 512, 1 << 20)
    assert e.value.status == B.ELAYOUT


def test_batched_pack_argument_errors():
    masks = B.rtoss_pattern_dict(2)
    good = (B.WDesc(32, 32, 3, 2, B.F16), 256, 512, 1024, 1 << 20)
    with pytest.raises(B.RtossError) as e:
        B.rtoss_pack_batch(None, masks)
    assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError) as e:  # second item: blob too small; nothing is launched
        B.rtoss_pack_batch([good, (B.WDesc(32, 32, 3, 2, B.F16), 256, 512, 1024, 16)], masks)
    assert e.value.status == B.ENOSPACE and "item 1" in str(e.value)
    with pytest.raises(B.RtossError) as e:  # dictionary / descriptor mismatch
        B.rtoss_pack_batch([(B.WDesc(32, 32, 3, 3, B.F16), 256, 512, 1024, 1 << 20)], masks)
    assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError) as e:
        B.rtoss_pack_batch([(B.WDesc(32, 32, 3, 2, B.F16), 0, 512, 1024, 1 << 20)], masks)
    assert e.value.status == B.EINVAL
    B.rtoss_pack_batch([], masks)



def test_coherent_path_argument_errors():
    masks = B.rtoss_pattern_dict(3)
    for bad in (B.WDesc(64, 32, 1, 3, B.F16), B.WDesc(64, 48, 3, 3, B.F16), B.WDesc(40, 32, 3, 3, B.F16),
                B.WDesc(64, 4096, 3, 3, B.F16), B.WDesc(64, 32, 3, 3, B.F32)):
        with pytest.raises(B.RtossError) as e:
            B.rtoss_pack_size_coherent(bad, masks)
        assert e.value.status == B.ESHAPE
    d = B.WDesc(64, 64, 3, 3, B.BF16)
    nbytes, off = B.rtoss_pack_size_coherent(d, masks)
    assert nbytes % 256 == 0 and off % 256 == 0 and nbytes >= off + 2 * 64 + 2 * 9 * 4096
    with pytest.raises(B.RtossError) as e:
        B.rtoss_pack_size_coherent(B.WDesc(64, 64, 3, 2, B.BF16), masks)  # k != popcount
    assert e.value.status == B.EINVAL
    with pytest.raises(B.RtossError) as e:
        B.rtoss_pack_coherent(d, 256, 512, masks, 1024, nbytes - 1)
    assert e.value.status == B.ENOSPACE
    with pytest.raises(B.RtossError) as e:
        B.rtoss_pack_coherent(d, 0, 512, masks, 1024, nbytes)
    assert e.value.status == B.EINVAL
    ok = B.CDesc(1, 8, 8, 1, 1, B.NHWC, B.BF16, 0)
    with pytest.raises(B.RtossError) as e:
        B.rtoss_conv2d_pattern_coherent(d, B.CDesc(1, 8, 8, 1, 1, B.NCHW, B.BF16, 0), None, masks, 256, 512, 1 << 20)
    assert e.value.status == B.ELAYOUT
    with pytest.raises(B.RtossError) as e:
        B.rtoss_conv2d_pattern_coherent(d, ok, None, masks, 0, 512, 1 << 20)
    assert e.value.status == B.EINVAL


@pytest.mark.parametrize("check", ["stem_rows_check", "share_check", "row_pieces_check", "work_order_check", "rows_cut_check"])
def test_index_arithmetic(tmp_path, check):
    """tests/<check>.cpp walks a header of the kernels on the CPU."""
    exe = str(tmp_path / check)
    subprocess.check_call([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-I", build.CSRC, os.path.join(ROOT, "tests", check + ".cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
