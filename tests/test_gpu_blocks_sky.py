"""Bins to the far side of the sky, where their chords crowd together: sets with the
largest chord tables (read from global memory), and just past them without one."""
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
