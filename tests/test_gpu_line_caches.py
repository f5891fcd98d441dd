"""The emit pass's line caches against the oracle: every per-line counter
exact, where the lines fit the workgroups' tables, where they overflow them
(pairs of slots taken by other lines, counted in global memory instead) and
where windows fill the staging of samples, copies and timers at once; the
shape for long single traces from 4,096 segments on, and the one below it and
for several traces in a launch."""
import pytest

import oracle
import tracegen as tg
from parity_util import compare

pytestmark = pytest.mark.gpu

SEG = 512
WIDE = 4096 * SEG  # events from which a single trace takes the wide shape


@pytest.fixture(scope="module")
def sampler():
    import paper_2212_07597_amd as smp
    s = smp.Sampler(workspace=4 << 30)
    yield s
    s.close()


def check(sampler, cases):
    import paper_2212_07597_amd as smp
    print("line caches:", len(cases), cases[0][0], flush=True)
    ids = [sampler.submit_trace(ev, smp.make_params(kw["threshold"], kw["num_lines"], kw["copy_threshold"]))
           for _, ev, kw in cases]
    sampler.run(blocking=True)
    for t, (label, ev, kw) in zip(ids, cases):
        compare(sampler.fetch_profile(t), oracle.run(ev, **kw), label)


@pytest.mark.parametrize("lines", [1, 700, 50_000])
@pytest.mark.parametrize("aux", [(0.02, 0.3), (0.6, 0.1), (0.95, 0.05)])
def test_counters(sampler, lines, aux):
    """Few to mostly copies and timers; a sample in most windows, or several."""
    cases = []
    for i, n in enumerate([SEG - 1, 40 * SEG + 7, WIDE - SEG, WIDE - SEG + 1, WIDE + 3 * SEG + 5]):
        ev = tg.mix(300 + i, n, num_lines=lines, copy_frac=aux[0], timer_frac=aux[1])
        for T in (tg.MiB // 64 + 1, 4 * tg.MiB):
            cases.append((f"n{n} L{lines} T{T} aux{aux}", ev,
                          dict(threshold=T, num_lines=lines, copy_threshold=100_003)))
    for c in cases:
        check(sampler, [c])
    check(sampler, cases)


@pytest.mark.parametrize("count", [319, 640, 1300])
def test_many_traces(sampler, count):
    """Runs of segments per trace: one round of workgroups, two, several."""
    ev = tg.mix(400, 20_000, num_lines=300, copy_frac=0.1, timer_frac=0.02)
    cases = []
    for i in range(count):
        n = [SEG - 1, 3 * SEG, 5 * SEG + 1, 9 * SEG + 17, 1][i % 5]
        cases.append((f"{count} traces, {i}", ev[i:i + n],
                      dict(threshold=tg.MiB // (1 << i % 4), num_lines=300, copy_threshold=100_003)))
    check(sampler, cases)


def test_emit_grids(sampler):
    """The default grid that a launch took is reported, written back it changes
    nothing, and a larger one set by the caller is taken as it is."""
    long = tg.mix(500, WIDE + 5, num_lines=60)
    one = [("one long trace", long, dict(threshold=tg.MiB, num_lines=60, copy_threshold=tg.MiB))]
    many = [(f"trace {i} of 1300", long[i:i + 700], one[0][2]) for i in range(1300)]
    try:
        sampler.set_tuning()
        short = sampler.get_tuning()["emit_grid"]
        for cases in (one, many):
            sampler.set_tuning()
            check(sampler, cases)
            took = sampler.get_tuning()["emit_grid"]
            assert took == short * 4 if cases is many else took < short
            sampler.set_tuning(emit_grid=took)
            check(sampler, cases)
            assert sampler.get_tuning()["emit_grid"] == took
        sampler.set_tuning(emit_grid=8 * short)
        check(sampler, one)
        assert sampler.get_tuning()["emit_grid"] == 8 * short
    finally:
        sampler.set_tuning()
