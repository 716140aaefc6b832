"""The block kernel's histogram and chord table share its LDS: edge sets on both
sides of each layout (table beside eight lane columns or more, table in global
memory with eight, four, two and one) give the oracle's counts, and a set with
fewer edges never takes much longer than one with more."""
import time

import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(c):
    return tuple(torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in c)


@pytest.mark.parametrize("mode", [pc.PC_MIXED, pc.PC_FP64_PLAIN])
@pytest.mark.parametrize("bins", [80, 90, 100, 125, 150, 200, 254, 400, 500, 700, 1000])
def test_counts_match_the_oracle(bins, mode):
    rng = np.random.default_rng(bins)
    patch = synth.centred_patch(12.0)
    A = synth.neyman_scott(320, 20, 0.05, patch, rng)
    B = synth.uniform_patch(4100, patch, rng)
    for n in (A[0].size, 900):                   # above and below 2^24 pairs
        a = tuple(x[:n] for x in A)
        for e in (synth.log_edges(0.01, 20.0, bins), synth.linear_edges(0.0, 9.0, bins)):
            got = pc.pc_count_ex(dev(a), e, B=dev(B), auto=False, mode=mode)
            assert got.tolist() == oracle.count(a, e, B=B, auto=False).tolist()


def test_fewer_bins_do_not_take_longer():
    """100,000 x 100,000 points: 150 bins took five times the time of 200 while
    their table was held in LDS beside a single column."""
    rng = np.random.default_rng(3)
    patch = synth.centred_patch(30.0)
    A, B = dev(synth.uniform_patch(100_000, patch, rng)), dev(synth.uniform_patch(100_000, patch, rng))

    def best(bins):
        e, t = synth.log_edges(0.01, 20.0, bins), []
        for _ in range(6):
            t0 = time.perf_counter()
            pc.pc_count(A, e, B=B, auto=False)
            t.append(time.perf_counter() - t0)
        return min(t)

    last = best(254)
    for bins in (200, 150, 125, 100, 80):
        t = best(bins)
        assert t < 1.5 * last, (bins, t, last)
        last = t
