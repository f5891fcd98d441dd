"""Tile maps (eight blocks of 64 segments built side by side, composed, and
chained while other tiles are built) against the oracle: traces that end
inside a block, tiles past the 32-bit range, tiles whose entries stay
unsampled too long for a map, and more tiles than one chaining step takes."""
import pytest

import oracle
import tracegen as tg
from parity_util import compare

pytestmark = pytest.mark.gpu

TILE = 512 * 512


@pytest.fixture(scope="module")
def sampler():
    import paper_2212_07597_amd as smp
    s = smp.Sampler(workspace=4 << 30)
    yield s
    s.close()


def check(sampler, ev, T, label, tiles=0):
    import paper_2212_07597_amd as smp
    print("tile maps:", label, flush=True)
    sampler.set_tuning(tile_map_tiles=tiles)
    try:
        tid = sampler.submit_trace(ev, smp.make_params(T, 40))
        sampler.run(blocking=True)
        c = sampler.last_counters()
        compare(sampler.fetch_profile(tid), oracle.run(ev, threshold=T, num_lines=40), label)
    finally:
        sampler.set_tuning()
    return c


@pytest.mark.parametrize("extra", [1, 512 * 63, 512 * 64, 512 * 64 + 1, 512 * 200 + 77])
def test_ragged_ends(sampler, extra):
    ev = tg.mix(91, 2 * TILE + extra, num_lines=40, copy_frac=0.05)
    c = check(sampler, ev, 64 * tg.MiB, f"2 tiles + {extra}", tiles=1)
    # (the short last tile may get none: a segment of one event has a constant
    # map, and entries still unsampled at its end leave more runs than a map holds)
    assert c[5] >= 2 and c[6] == c[5]


def test_past_32_bits(sampler):
    """Thresholds at and past 2^30: the tiles take the 64-bit path."""
    ev = tg.mix(92, 2 * TILE + 5000, num_lines=40, size_lo=1 << 14, size_hi=1 << 25)
    for T in (1 << 30, (1 << 32) + 1):
        check(sampler, ev, T, f"T {T}", tiles=1)
    ev = tg.mix(93, 2 * TILE + 5000, num_lines=40, size_lo=1 << 20, size_hi=1 << 28)
    check(sampler, ev, 1 << 35, "steps past 2^30 in a segment", tiles=1)


def test_many_tiles(sampler):
    """By default from 8 tiles on; 70 tiles chain in more than one step."""
    ev = tg.mix(94, 70 * TILE + 3, num_lines=40)
    c = check(sampler, ev, 48 * tg.MiB, "71 tiles")
    assert c[5] >= 70 and c[6] >= 70
    c = check(sampler, ev[:8 * TILE], 400 * tg.MiB, "entries unsampled too long for a map")
    assert c[6] <= 8


def test_maps_are_built(sampler):
    """The cases above reach the paths that they are about: the 64-bit build
    (all of these tiles need it) and the refusal before a build."""
    ev = tg.mix(92, 2 * TILE + 5000, num_lines=40, size_lo=1 << 14, size_hi=1 << 25)
    c = check(sampler, ev, 1 << 30, "T at 2^30, built", tiles=1)
    assert c[5] >= 2 and c[6] == c[5]
    ev = tg.mix(93, 2 * TILE + 5000, num_lines=40, size_lo=1 << 20, size_hi=1 << 28)
    c = check(sampler, ev, 1 << 35, "steps past 2^30 in a segment, built", tiles=1)
    assert c[5] >= 2 and c[6] == c[5]
    ev = tg.mix(94, 8 * TILE, num_lines=40)
    c = check(sampler, ev, 400 * tg.MiB, "refused")
    assert c[5] == 0 and c[6] == 0 and c[8] == 8
    c = check(sampler, ev, 2 * tg.MiB, "segments that move T or more")
    assert c[5] == 0 and c[7] == 8
