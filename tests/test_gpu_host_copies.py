"""Host catalogues of a call go to the device in one copy up to 96 x 1024
values together and array by array beyond: equal counts on both sides of the
line, with device catalogues between them, repeated ones, row ranges, and an
invalid point in either."""
import numpy as np
import pytest

import paper_1208_3658_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

E = synth.log_edges(0.01, 3.0, 11)


@pytest.mark.parametrize("n,m", [(1, 2), (700, 1301), (24576, 24576), (24577, 24576), (60000, 5)])
def test_both_sides_of_the_line(n, m):
    rng = np.random.default_rng(n)
    patch = synth.centred_patch(15.0)
    A, B, C = (synth.uniform_patch(k, patch, rng) for k in (n, m, 900))
    dA, dB, dC = (tuple(torch.from_numpy(x).cuda() for x in c) for c in (A, B, C))
    jobs = lambda a, b: [{"A": a, "edges": E}, {"A": a, "B": b, "edges": E, "auto": False},
                         {"A": dC, "B": b, "edges": E, "auto": False}, {"A": b, "edges": E},
                         {"A": a, "edges": E, "rows": (n // 3, n - n // 4)}]
    for mode in (pc.PC_MIXED, pc.PC_FP64_PLAIN):
        want = [c.tolist() for c in pc.pc_count_batch(jobs(dA, dB), mode=mode)]
        assert [c.tolist() for c in pc.pc_count_batch(jobs(A, B), mode=mode)] == want
        assert [c.tolist() for c in pc.pc_count_batch_static(jobs(A, B), mode=mode)] == want
    bad = (B[0], B[1].copy())
    bad[1][-1] = np.nan
    with pytest.raises(pc.PcError) as e:
        pc.pc_count_batch(jobs(A, bad))
    assert e.value.code == pc.PC_ERR_INVALID
