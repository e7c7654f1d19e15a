"""The automatic z-chunk of the fused DUGKS step attains the least estimated cost
over every candidate, plain and cut (host computation, no GPU needed)."""
import math

import pytest

import paper_1601_03815_amd as dhit


def _candidates(n, tile, slots):
    """Cost of each signed chunk (negative: the last round cut), from the rules
    of the z_chunk field: chunks ceil(n/k) of at least min(n, 8) planes, and
    shorter ones whose items fit one round (at most 1024); a launch costs its
    rounds times (planes + 2), a cut one its full rounds and one of parts.
    A last round of t chunks is cut into ceil(c/len) parts of len =
    ceil(c / min(slots // t, c)) planes when it fills at most half a round
    behind at least one full one."""
    tiles = math.ceil(n / (tile - 2)) * math.ceil(n / 6)
    cost = {}
    for c in {math.ceil(n / k) for k in range(1, n + 1)}:
        blocks = tiles * math.ceil(n / c)
        if c < min(n, 8) and blocks > min(slots, 1024):
            continue
        cost[c] = math.ceil(blocks / slots) * (c + 2)
        full, t = divmod(blocks, slots)
        if full and t and min(slots // t, c) >= 2:
            length = math.ceil(c / min(slots // t, c))
            parts = math.ceil(c / length)
            if parts > 1:
                cost[-c] = full * (c + 2) + math.ceil(c / parts) + 2
    return cost


@pytest.mark.parametrize("n", [4, 7, 9, 16, 24, 32, 33, 40, 48, 49, 64, 80, 97, 128, 160, 225, 256])
@pytest.mark.parametrize("tile", [16, 32])
@pytest.mark.parametrize("slots", [64, 256, 512, 1024, 4096])
def test_automatic_choice_is_the_cheapest(n, tile, slots):
    p = dhit.default_params(n, dhit.DUGKS, dhit.FP64, 0.01)
    p.tile_width = tile
    zc = dhit.fused_work_items(p, slots)[1]
    cost = _candidates(n, tile, slots)
    best = min(cost.values())
    assert cost[zc] == best
    # of equal ones the longest, and the uncut one
    assert max((abs(c), c > 0) for c in cost if cost[c] == best) == (abs(zc), zc > 0)


def test_cut_choices_occur():
    """The sizes above exercise both kinds."""
    cut = sum(min(c, key=lambda k: (c[k], -abs(k), k < 0)) < 0
              for n in (33, 64, 97, 128, 160, 225, 256) for t in (16, 32) for s in (64, 256, 512)
              for c in [_candidates(n, t, s)])
    assert 5 < cut < 40
