"""Block maps of the resolve pass (64 segments of 512 events followed for all
entries at once) against the oracle: every output exact, as everywhere.

The sizes are the edges of segments, blocks and tiles; the thresholds go from
many samples in a segment to entries that stay unsampled past the block's
limit (the tile is walked instead), and past the 32-bit range of the maps."""
import numpy as np
import pytest

import oracle
import tracegen as tg
from parity_util import compare

pytestmark = pytest.mark.gpu

SEG, BLK, TILE = 512, 64 * 512, 512 * 512


@pytest.fixture(scope="module")
def sampler():
    import paper_2212_07597_amd as smp
    s = smp.Sampler(workspace=4 << 30)
    yield s
    s.close()


def check(sampler, cases):
    import paper_2212_07597_amd as smp
    print("block maps:", [c[0] for c in cases], flush=True)
    ids = [sampler.submit_trace(ev, smp.make_params(kw["threshold"], kw["num_lines"], kw.get("copy_threshold")))
           for _, ev, kw in cases]
    sampler.run(blocking=True)
    for t, (label, ev, kw) in zip(ids, cases):
        compare(sampler.fetch_profile(t), oracle.run(ev, **kw), label)


@pytest.mark.parametrize("T", [tg.MiB // 2 + 1, 2 * tg.MiB, 3 * tg.MiB + 1, 10 * tg.MiB, 24 * tg.MiB, 40 * tg.MiB])
def test_sizes(sampler, T):
    """Block and tile edges, alone and in one launch."""
    ev = tg.mix(77, 2 * TILE + BLK + 300, num_lines=50, copy_frac=0.05, timer_frac=0.01)
    sizes = [7 * SEG, 8 * SEG, 9 * SEG + 1, BLK - 1, BLK, BLK + 1, BLK + SEG + 3, 5 * BLK + 31, TILE, TILE + 20,
             2 * TILE + BLK + 300]
    cases = [(f"n{n} T{T}", ev[:n], dict(threshold=T, num_lines=50)) for n in sizes]
    check(sampler, cases)
    for c in cases[-3:]:
        check(sampler, [c])


def test_mixed_segments(sampler):
    """Segments every entry samples in, segments with one exit and segments
    that depend on the entry, side by side; a footprint that drifts; sizes up
    to and past the 32-bit range of the maps."""
    rng = np.random.default_rng(5)
    n = 3 * BLK + 1000
    base = tg.mix(78, n, num_lines=9)
    forced = base.copy()
    at = rng.choice(n, 40, replace=False)
    forced["delta"][at] = np.where(rng.random(40) < 0.5, 1, -1) * 25 * tg.MiB
    forced["flags"][at] = 1
    quiet = base.copy()  # stretches of small steps between loud ones
    quiet["delta"][(np.arange(n) // 3000) % 2 == 1] //= 64
    wide = tg.mix(79, n, num_lines=9, size_lo=1 << 20, size_hi=1 << 27)
    edge = tg.mix(80, n, num_lines=9, size_lo=1 << 10, size_hi=1 << 20)
    edge["delta"][::7000] = (1 << 30) - 7
    edge["delta"][3::7000] = -(1 << 30) + 7
    cases = [("forced", forced, 10 * tg.MiB), ("forced small T", forced, 3 * tg.MiB), ("quiet", quiet, 10 * tg.MiB),
             ("quiet small T", quiet, 2 * tg.MiB), ("wide", wide, (1 << 29) + 1), ("wide below", wide, (1 << 30) - 1),
             ("wide at", wide, 1 << 30), ("edge", edge, 10 * tg.MiB), ("edge high", edge, (1 << 30) - 1)]
    check(sampler, [(label, ev, dict(threshold=T, num_lines=9)) for label, ev, T in cases])


def test_still_segments(sampler):
    """Segments that move less than T, whose map comes from their extremes:
    one extreme reached at once (constant exit), reached by steps, on both
    sides, from the other side first, and no movement at all."""
    def trace(*segments):
        d = np.zeros(len(segments) * SEG, np.int64)
        for i, steps in enumerate(segments):
            for at, x in steps:
                d[i * SEG + at] = x
        ev = np.zeros(d.shape[0], dtype=tg.EVENT_DTYPE)
        ev["delta"] = d
        ev["ptr"] = np.arange(1, d.shape[0] + 1)
        ev["line"] = np.arange(d.shape[0]) % 5
        return ev
    shapes = [[(0, 40)], [(511, 40)], [(3, 40), (70, -10)], [(3, 40), (70, -45)], [(3, -30)], [(3, -30), (90, 55)],
              [(9, 20), (400, 20)], [(9, 20), (80, -20), (300, 20)], [(5, 1)], [(5, -1)], [], [(64, 99)], [(63, -99)],
              [(0, 50), (1, -100)], [(0, 49), (1, -99), (2, 99)]]
    rng = np.random.default_rng(4)
    order = [shapes[i] for i in rng.integers(0, len(shapes), 300)]
    cases = [(f"still T{T}", trace(*order), dict(threshold=T, num_lines=5)) for T in (50, 100, 101, 150, 1000)]
    check(sampler, cases)


@pytest.mark.parametrize("segments", [8, 9, 20, 63, 64, 65, 130])
def test_workspace_without_room_to_spare(segments):
    """A trace of a few blocks alone in a workspace of exactly its size."""
    import paper_2212_07597_amd as smp
    import torch
    n = segments * SEG - 100
    ev = tg.mix(85, n, num_lines=20)
    dev = torch.from_numpy(ev.view(np.uint8)).to("cuda")
    p = smp.make_params(2 * tg.MiB, 20)
    with_room = smp.sampler_fixed_bytes() + smp.workspace_bytes(n, p, ev_on_device=True)
    s = smp.Sampler(workspace=with_room)
    try:
        print("exact workspace:", segments, flush=True)
        tid = s.submit_trace(dev, p)
        s.run(blocking=True)
        compare(s.fetch_profile(tid), oracle.run(ev, threshold=2 * tg.MiB, num_lines=20), f"{segments} segments")
    finally:
        s.close()


def counted(sampler, ev, T, label):
    """(tiles resolved through block maps, tiles whose maps did not fit)."""
    check(sampler, [(label, ev, dict(threshold=T, num_lines=50))])
    return tuple(sampler.last_counters()[11:13])


@pytest.mark.parametrize("n,maps", [(2 * BLK, 1), (2 * BLK + 1, 1), (3 * BLK - 1, 1), (3 * BLK, 1), (3 * BLK + 1, 1),
                                    (5 * BLK + 31, 1), (TILE - 1, 1), (TILE, 1), (TILE + 8 * SEG, 2),
                                    (TILE + 9 * SEG + 1, 2), (TILE + BLK - 1, 2), (TILE + BLK + 1, 2),
                                    (2 * TILE + BLK + 300, 3)])
def test_maps_are_taken(sampler, n, maps):
    """Block and tile edges where the maps are what gives the result."""
    ev = tg.mix(77, n, num_lines=50, copy_frac=0.05, timer_frac=0.01)
    assert counted(sampler, ev, 3 * tg.MiB, f"maps at n{n}") == (maps, 0)


def test_maps_that_are_not_taken(sampler):
    """Short walks, chains that do not fit and thresholds past the 32-bit range."""
    ev = tg.mix(77, 2 * TILE + BLK + 300, num_lines=50, copy_frac=0.05, timer_frac=0.01)
    assert counted(sampler, ev[:BLK], 10 * tg.MiB, "one block, walked") == (0, 0)
    assert counted(sampler, ev[:TILE], 30 * tg.MiB, "few stops, walked") == (0, 0)
    taken, given_up = counted(sampler, ev, 30 * tg.MiB, "second tile's chains do not fit")
    assert given_up >= 1
    wide = tg.mix(79, 3 * BLK, num_lines=50, size_lo=1 << 20, size_hi=1 << 27)
    assert counted(sampler, wide, 1 << 30, "threshold past the range") == (0, 0)
