"""The rate-based sampler's tiles (8 or 16 segments of 512 events, by the
trace's length) against the oracle: sizes around a tile, around the length
where tiles grow and around a look-back of 64 tiles, thresholds from every
byte a sample to the largest, and errors that a late tile finds."""
import numpy as np
import pytest

import oracle
import tracegen as tg

pytestmark = pytest.mark.gpu

SMALL, LARGE, GROW = 8 * 512, 16 * 512, 512 << 10


def check(ev, T, L, label):
    import paper_2212_07597_amd as smp
    import torch
    print("rate tiles:", label, flush=True)
    st, K, counts = smp.rate_run(torch.from_numpy(ev.view(np.uint8)).to("cuda"), T, L)
    ost, oK, ocounts = oracle.rate(ev, T, L)
    assert st == ost, (label, st, ost)
    if ost == oracle.OK:
        assert K == oK, (label, K, oK)
        np.testing.assert_array_equal(counts, ocounts, err_msg=label)


@pytest.mark.parametrize("n", [SMALL - 1, SMALL, SMALL + 1, 65 * SMALL + 3, GROW - 1, GROW, GROW + 1, 66 * LARGE,
                               66 * LARGE + 4097, 600 * LARGE + 5])
def test_sizes(n):
    ev = tg.mix(n % 11, n, num_lines=300, copy_frac=0.03, timer_frac=0.01)
    for T in (1, 12_345, 10 << 20, (1 << 60) - 1):
        check(ev, T, 300, f"n={n} T={T}")


@pytest.mark.parametrize("n", [3 * SMALL, GROW + 3 * LARGE])
def test_errors_in_the_last_tile(n):
    ev = tg.mix(3, n, num_lines=20)
    bad = ev.copy()
    bad["line"][n - 1] = 20
    check(bad, 1 << 20, 20, f"malformed n={n}")
    big = ev.copy()
    big["delta"][-1100:] = np.where(np.arange(1100) % 2 == 0, 1, -1) * ((1 << 52) - 1)
    big["flags"][-1100:] = 0
    check(big, 1 << 20, 20, f"overflow n={n}")
    big["line"][5] = 99
    check(big, 1 << 20, 20, f"malformed and overflow n={n}")


@pytest.mark.parametrize("n,size", [(GROW + 3 * LARGE, LARGE), (GROW, SMALL)])
def test_volumes_past_64_bits_in_a_tile(n, size):
    """Tiles whose volume is 2^64 and a little more (2^63 for the small ones),
    or 2^65 and a little less; first, in the middle and the last whole one."""
    ev = tg.mix(4, n, num_lines=20)
    last = n // size - 1
    for tile in (0, last // 2, last):
        for d in ((1 << 51), (1 << 51) + 12_345, (1 << 51) + (1 << 49) - 1, (1 << 52) - 1):
            big = ev.copy()
            big["delta"][tile * size:(tile + 1) * size] = np.where(np.arange(size) % 2 == 0, 1, -1) * d
            big["flags"][tile * size:(tile + 1) * size] = 0
            assert oracle.rate(big, 1 << 20, 20)[0] == oracle.EOVERFLOW
            check(big, 1 << 20, 20, f"n={n} tile {tile} delta {d}")
    # the largest total that still counts (2^62 - 1) and the smallest that does not, in one tile and spread out
    for at in (np.arange(1100), np.linspace(0, n - 1, 1100).astype(int)):
        for total in ((1 << 62) - 1, 1 << 62):
            edge = ev.copy()
            edge["delta"], edge["flags"] = 0, 0
            edge["delta"][at] = total // 1100
            edge["delta"][at[:total % 1100]] += 1
            assert int(edge["delta"].sum(dtype=np.uint64)) == total
            check(edge, 1 << 40, 20, f"n={n} total {total}")
