"""Edge sets of many bins on a field about as wide as the last edge: most blocks
meet several edges and go through the chord table, mixed launches hold it in LDS
with three workgroups a CU, and binary64 takes pairs that are none back from the
table's first row.  Counts equal the oracle's, ragged and diagonal blocks among
them."""
import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SETS = {"log_100": synth.log_edges(0.5, 30.0, 100), "log_170": synth.log_edges(0.5, 30.0, 170),
        "log_250": synth.log_edges(0.1, 30.0, 250), "even_40": synth.linear_edges(0.0, 30.0, 40),
        "even_100": synth.linear_edges(0.0, 20.0, 100)}


def dev(c):
    return tuple(torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in c)


@pytest.mark.parametrize("mode", [pc.PC_MIXED, pc.PC_FP64_PLAIN])
@pytest.mark.parametrize("kind", sorted(SETS))
def test_counts(kind, mode):
    e = SETS[kind]
    rng = np.random.default_rng(61)
    patch = synth.centred_patch(50.0)
    B = synth.uniform_patch(3001, patch, rng)
    for n in (6001, 6143, 37):                   # above, above and below 2^24 pairs; 17, 31 and 5 points in the last group
        A = synth.uniform_patch(n, patch, rng)
        assert pc.pc_count_ex(dev(A), e, mode=mode).tolist() == oracle.count(A, e).tolist()
        got = pc.pc_count_ex(dev(A), e, B=dev(B), auto=False, mode=mode)
        assert got.tolist() == oracle.count(A, e, B=B, auto=False).tolist()
