"""Bins to the far side of the sky, where their chords crowd together: sets with the
largest chord tables (read from global memory), and just past them without one;
and small calls in many wide bins."""
import time

import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def sky(n, rng):
    return 360.0 * rng.random(n), np.degrees(np.arcsin(2.0 * rng.random(n) - 1.0))


def dev(c):
    return tuple(torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in c)


@pytest.mark.parametrize("mode", [pc.PC_MIXED, pc.PC_FP64_PLAIN])
@pytest.mark.parametrize("bins", [60, 100, 179, 180, 400])
def test_counts_match_the_oracle(bins, mode):
    rng = np.random.default_rng(bins)
    A, B = sky(6001, rng), sky(4099, rng)
    for e in (synth.linear_edges(0.0, 180.0, bins), synth.linear_edges(100.0, 178.0, bins)):
        for n in (6001, 117):                    # above and below 2^24 pairs
            a = tuple(x[:n] for x in A)
            assert pc.pc_count_ex(dev(a), e, B=dev(B), auto=False, mode=mode).tolist() == oracle.count(a, e, B=B, auto=False).tolist()
            assert pc.pc_count_ex(dev(a), e, auto=True, mode=mode).tolist() == oracle.count(a, e, auto=True).tolist()


@pytest.mark.parametrize("bins", [150, 200, 254, 300])
def test_counts_of_small_calls_match_the_oracle(bins):
    rng = np.random.default_rng(bins)
    for n in (64, 513, 2000):
        A = sky(n, rng)
        for e in (synth.linear_edges(36.0, 123.0, bins), synth.log_edges(0.1, 60.0, bins)):
            assert pc.pc_count(dev(A), e).tolist() == oracle.count(A, e, auto=True).tolist()


def test_small_calls_take_many_bins_as_they_take_few():
    """3000 points on the whole sky: 300 bins took four times the time of 60 with the
    two columns that four workgroups a CU leave beside the table, and 1.2 times with
    eight."""
    A = dev(sky(3000, np.random.default_rng(5)))

    def best(bins):
        e, t = synth.linear_edges(36.9, 123.0, bins), []
        for _ in range(12):
            t0 = time.perf_counter()
            pc.pc_count(A, e)
            t.append(time.perf_counter() - t0)
        return min(t)

    assert best(300) < 2.0 * best(60)
