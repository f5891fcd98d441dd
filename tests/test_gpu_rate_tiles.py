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
