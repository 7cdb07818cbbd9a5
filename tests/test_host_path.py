"""The native call path behind pipeline.py: its own argument checks, what it holds on to during a call, and layers as
ordinary Python objects (no GPU needed)."""
import copy
import pickle
import subprocess
import sys

import numpy as np
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl

from conftest import ROOT


@pytest.fixture
def layer():
    return pl.PackedLayer(32, 32, 3, 3, B.F16, B.rtoss_pattern_dict(3), device="cpu")


def test_arguments_are_checked_before_the_library_is_called(layer):
    x = torch.zeros(1, 4, 4, 32, dtype=torch.float16)
    with pytest.raises(AssertionError):
        layer.conv(x)  # not on the GPU
    with pytest.raises(AssertionError):
        layer.conv_fused(x)
    with pytest.raises(TypeError):
        layer.conv(np.zeros((1, 4, 4, 32), np.float16))
    with pytest.raises(AssertionError):
        pl.select_patterns(torch.zeros(32, 32, 3, 3), B.F32, layer.masks)
    with pytest.raises(AssertionError):
        pl.pack_layers([layer], [torch.zeros(32, 32, 3, 3)], [torch.zeros(1024, dtype=torch.uint8)])
    assert pl.pack_layers([], [], []) == []


def test_library_errors_carry_status_and_message():
    with pytest.raises(B.RtossError) as e:
        pl.select_patterns_batch([], 7, B.rtoss_pattern_dict(3), stream=0)
    assert e.value.status == B.EDTYPE and "dtype" in str(e.value)
    # dictionaries of other integer types are converted, as everywhere in the binding
    assert pl.select_patterns_batch([], B.F16, B.rtoss_pattern_dict(3).astype(np.int64), stream=0) == []


LISTS_CHANGED_DURING_A_CALL = """
import threading, time, torch
from torch._subclasses.fake_tensor import FakeTensorMode
from paper_2303_02191_amd import binding as B, pipeline as pl

masks = B.rtoss_pattern_dict(3)
with FakeTensorMode():  # empty tensors that say they are on a GPU: the library has nothing to launch for them
    w, idx = torch.empty(0, dtype=torch.float16, device="cuda"), torch.empty(0, dtype=torch.uint8, device="cuda")
n = 300000
ws, idxs, inside = [w] * n, [idx] * n, threading.Event()

class Dtype:
    def __index__(self):  # converted inside the call
        inside.set()
        return B.F16

def shorten():
    inside.wait()
    time.sleep(0.001)  # gets to run when the call gives up the interpreter lock
    idxs.clear()
    ws.clear()

thread = threading.Thread(target=shorten)
thread.start()
out = B.host().select_batch(ws, Dtype(), masks, idxs, 0)
thread.join()
assert len(out) in (0, n) and len(ws) == 0  # (0: a loaded machine let the other thread run before the call had its copy)

# an attribute of a layer that runs Python code and shortens the lists of the call
layer = pl.PackedLayer(32, 32, 3, 3, B.F16, masks, device="cpu")
layers, ws, idxs = [], [torch.zeros(32, 32, 3, 3)] * 3, [torch.zeros(1024, dtype=torch.uint8)] * 3

class Shortening:
    blob = layer.blob

    @property
    def _native(self):
        layers.clear()
        ws.clear()
        idxs.clear()
        return layer._native

layers += [Shortening(), Shortening(), Shortening()]
try:
    B.host().pack_batch(layers, ws, idxs, 0)
except AssertionError:  # (weights on the CPU)
    print("survived")
"""


def test_lists_that_change_during_a_call():
    """The call works on the elements its lists had when it began.  (In a process of its own: reading past a shortened
    list ends it.)"""
    p = subprocess.run([sys.executable, "-c", LISTS_CHANGED_DURING_A_CALL], capture_output=True, text=True, timeout=300,
                       cwd=ROOT)
    assert p.returncode == 0 and "survived" in p.stdout, (p.returncode, p.stderr[-2000:])


KINDS = [lambda masks, device="cpu": pl.PackedLayer(32, 32, 3, 3, B.F16, masks, device=device),
         lambda masks, device="cpu": pl.CoherentLayer(32, 32, 3, B.F16, masks, device=device)]


def refusal(layer):
    """What the library says to packing the layer from tensors without memory: the descriptor and the dictionary are looked
    at before the pointers."""
    with FakeTensorMode():
        w = torch.empty(32, 32, 3, 3, dtype=torch.float16, device="cuda")
        idx = torch.empty(1024, dtype=torch.uint8, device="cuda")
    with pytest.raises(B.RtossError) as e:
        pl.pack_layers([layer], [w], [idx], stream=0)
    return str(e.value)


@pytest.mark.parametrize("make", KINDS)
def test_layers_can_be_copied_and_pickled(make):
    layer = make(B.rtoss_pattern_dict(3))
    layer.blob.random_(0, 255)
    for other in (copy.copy(layer), copy.deepcopy(layer), pickle.loads(pickle.dumps(layer))):
        assert type(other) is type(layer) and other.packed_bytes == layer.packed_bytes and other.dt == layer.dt
        assert bytes(other.wdesc) == bytes(layer.wdesc) and np.array_equal(other.masks, layer.masks)
        assert torch.equal(other.blob, layer.blob)
        assert "taps" not in refusal(other)
        other.masks = B.rtoss_pattern_dict(2)  # its own from here on
        assert "dictionary keeps 2 taps" in refusal(other) and "taps" not in refusal(layer)


@pytest.mark.parametrize("make", KINDS)
def test_calls_follow_a_layers_attributes(make):
    masks = B.rtoss_pattern_dict(3)
    layer = make(masks)
    assert "taps" not in refusal(layer)
    layer.wdesc.k = 2  # in place
    assert "dictionary keeps 3 taps, descriptor says k=2" in refusal(layer)
    layer.wdesc = B.WDesc(32, 32, 3, 3, B.F16)
    assert "taps" not in refusal(layer)
    masks[1] = 3  # in place
    assert "pattern 1 keeps 2 taps" in refusal(layer)
    layer.masks = [7, 0x1c0]  # any sequence
    assert "taps" not in refusal(layer)
    layer.masks.append(3)
    assert "pattern 2 keeps 2 taps" in refusal(layer)


def test_a_layer_of_another_build_in_host_memory_reaches_no_kernel():
    """Its private sections would be read as today's: calls refuse it until its blob is on a GPU, where it is packed again.  (Of another
    build: without the mark of today's sections, and of another size.)"""
    layer = pl.PackedLayer(64, 96, 3, 5, B.BF16, B.rtoss_pattern_dict(5), device="cpu")
    state = layer.__getstate__()
    del state["private_format"]
    kept = pl.PackedLayer.__new__(pl.PackedLayer)
    kept.__setstate__(dict(state))
    assert "taps" not in refusal(kept) and kept.blob is layer.blob  # the same size: the same sections
    old = pl.PackedLayer.__new__(pl.PackedLayer)
    old.__setstate__(dict(state, blob=torch.zeros(layer.packed_bytes + 512, dtype=torch.uint8)))
    later = pl.PackedLayer.__new__(pl.PackedLayer)
    later.__setstate__(dict(state, private_format=pl.PackedLayer.PRIVATE_FORMAT + 1))
    for other in (old, copy.copy(old), pickle.loads(pickle.dumps(old)), later):
        other.masks = list(other.masks)
        with FakeTensorMode():
            x = torch.empty(1, 4, 4, 96, dtype=torch.bfloat16, device="cuda")
        for call in (lambda: other.conv(x), lambda: other.conv_fused(x), lambda: refusal(other)):
            with pytest.raises(RuntimeError, match="another build"):
                call()
    assert layer.private_format == pl.PackedLayer.PRIVATE_FORMAT and copy.copy(layer).private_format == layer.private_format


@pytest.mark.gpu
@pytest.mark.parametrize("make", KINDS)
def test_copies_compute_and_follow_their_attributes(make):
    masks = B.rtoss_pattern_dict(3)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    w = torch.randn((32, 32, 3, 3), generator=g, device="cuda").half()
    x = torch.randn((1, 9, 11, 32), generator=g, device="cuda").half()
    layer = make(masks, "cuda").pack(w, pl.select_patterns(w, B.F16, masks))
    y = layer.conv(x)
    for other in (copy.copy(layer), copy.deepcopy(layer), pickle.loads(pickle.dumps(layer))):
        assert torch.equal(other.conv(x), y)
        other.dt = B.F32  # the default type of results
        assert other.conv(x).dtype == torch.float32
        other.masks = list(masks)
        other.dt = B.F16
        assert torch.equal(other.conv(x), y)
        other.masks = B.rtoss_pattern_dict(2)
        with pytest.raises(B.RtossError):
            other.conv(x)
    assert torch.equal(layer.conv(x), y)
