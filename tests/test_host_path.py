"""The native call path behind pipeline.py: its own argument checks, what it holds on to during a call, and layers as
ordinary Python objects (no GPU needed)."""
import subprocess
import sys

import numpy as np
import pytest
import torch

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
assert len(out) == n and len(ws) == 0

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
