"""Which dictionaries the 2-of-4 steps take, by the size of the packed section: a search of its own over every way to give a pattern's taps
to the groups, for single patterns and for the dictionaries of every size and rule."""
import itertools

import numpy as np
import pytest

from paper_2303_02191_amd import binding as B

GROUPS = [(0, 4, 8, 7), (1, 5, 6, 8), (2, 3, 7, 5)]  # (the last tap of each stands in another group too)
Co, Ci = 128, 96


def places(mask, groups):
    """At most two taps a group, every tap in one of its groups."""
    taps = [[g for g, members in enumerate(groups) if t in members] for t in range(9) if mask >> t & 1]
    return any(max(choice.count(g) for g in set(choice)) <= 2 for choice in itertools.product(*taps))


def expected(masks):
    corners, edges = 0b101000101, 0b010101010
    if all(bin(m & corners).count("1") <= 2 and bin(m & edges).count("1") <= 2 for m in masks):
        return 5 * 1024 + 2 * 256
    if all(places(m, [g[:3] for g in GROUPS]) for m in masks):
        return 6 * 1024 + 3 * 256
    # (where a tap is needed in its second group: the dense fragments as well)
    return 6 * 1024 + 3 * 256 + 9 * 1024 if all(places(m, GROUPS) for m in masks) else 9 * 1024


def tile_bytes(masks):
    k = bin(masks[0]).count("1")
    groups = Co * Ci
    size, _ = B.rtoss_pack_size(B.WDesc(Co, Ci, 3, k, B.F16), np.array(masks, dtype=np.uint16))
    public = -(-groups * k * 2 // 256) * 256 + groups
    return (size - public) // (Ci // 32 * Co // 16)  # (the block of zeros at the end is less than a byte a tile's share)


def test_every_pattern():
    got = {m: tile_bytes([m]) for m in range(1, 512)}
    want = {m: expected([m]) for m in range(1, 512)}
    assert {m: (g, want[m]) for m, g in got.items() if not want[m] <= g < want[m] + 64} == {}
    assert sum(v == 9 * 1024 for v in want.values()) == 60  # 451 of the 511 are placed


@pytest.mark.parametrize("rule", [B.RULE_ALL, B.RULE_ANYPAIR4, B.RULE_CONNECTED4, B.RULE_CONNECTED8])
def test_dictionaries(rule):
    for k in range(1, 10):
        masks = [int(m) for m in B.rtoss_pattern_dict(k, rule)]
        if not 1 <= len(masks) <= 255:
            continue
        assert expected(masks) <= tile_bytes(masks) < expected(masks) + 64, k
    masks = [int(m) for m in B.rtoss_pattern_dict(5, B.RULE_CONNECTED4)]
    assert expected(masks) == 6 * 1024 + 3 * 256 + 9 * 1024
