"""The native call path behind pipeline.py: its own argument checks (no GPU needed)."""
import numpy as np
import pytest
import torch

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl


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
