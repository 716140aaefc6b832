"""The spatial ordering takes its views in rounds where their counters do not fit
the region they have: batches of many views, ordinary and in the fixed area,
count what each catalogue counts by itself."""
import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

E = synth.log_edges(0.02, 5.0, 20)


def catalogues(count, n):
    rng = np.random.default_rng(count)
    patch = synth.centred_patch(10.0)
    ra, dec = synth.uniform_patch(count * n, patch, rng)
    d = tuple(torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (ra, dec))
    cats = [(ra[k * n:(k + 1) * n], dec[k * n:(k + 1) * n]) for k in range(count)]
    return cats, [tuple(x[k * n:(k + 1) * n] for x in d) for k in range(count)]


@pytest.mark.parametrize("count,n,mode,static", [
    (1100, 4000, pc.PC_MIXED, False),                          # 70 MB of counters: two rounds
    (2600, 1000, pc.PC_MIXED, True), (2600, 1000, pc.PC_MIXED | pc.PC_MATRIX_CORES, True),
    (540, 5000, pc.PC_MIXED | pc.PC_MATRIX_CORES, True), (700, 5003, pc.PC_FP64_PLAIN, True)])
def test_many_views(count, n, mode, static):
    cats, devs = catalogues(count, n)
    jobs = [{"A": a, "edges": E} for a in devs]
    got = (pc.pc_count_batch_static if static else pc.pc_count_batch)(jobs, mode=mode)
    want = [pc.pc_count(a, E) for a in devs]
    for k, (g, w) in enumerate(zip(got, want)):
        assert g.tolist() == w.tolist(), k
    for k in (0, count // 2, count - 1):
        assert got[k].tolist() == oracle.count(cats[k], E).tolist(), k


def test_an_ordinary_call_allocates_the_survivors_it_can_write():
    """300,000 x 300,000 points: 32 bytes a point converted, 53 ordered, 16 for the
    ordering's counters, whose place the survivors of 586 x 586 pairs of 512-point
    tiles take (16 bytes each, 5.5 MB; 22 MB for pairs of 256-point tiles)."""
    cats, devs = catalogues(2, 300_000)
    got = pc.pc_count(devs[0], E, B=devs[1], auto=False)
    assert pc.pc_debug_last_workspace() < 102 * 600_000
    assert got.tolist() == pc.pc_count_ex(devs[0], E, B=devs[1], auto=False, mode=pc.PC_FP64_PLAIN).tolist()
