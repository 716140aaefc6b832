"""Calls of few pairs are counted in the caller's order, without the spatial
ordering: counts equal the oracle's on both sides of the line (2^24 pairs of a
call), for tiles that span the whole sky, for catalogues sorted against the
blocks, and in batches whose pairs add up."""
import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LOG, EVEN = synth.log_edges(0.003, 60.0, 33), synth.linear_edges(0.0, 9.0, 18)


def dev(c):
    return tuple(torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in c)


def sky(n, rng):
    return 360.0 * rng.random(n), np.degrees(np.arcsin(2.0 * rng.random(n) - 1.0))


@pytest.mark.parametrize("n,m", [(2, 1), (33, 700), (5792, 2896), (5793, 2897), (4096, 4096), (4096, 4097)])
@pytest.mark.parametrize("where", ["sky", "patch", "clustered", "sorted"])
def test_both_sides_of_the_line(n, m, where):
    rng = np.random.default_rng(n + m)
    if where == "sky":
        A, B = sky(n, rng), sky(m, rng)
    elif where == "clustered":
        patch = synth.centred_patch(12.0)
        A, B = (synth.neyman_scott(k // 20 + 1, 20, 0.02, patch, rng) for k in (n, m))
    else:
        patch = synth.centred_patch(25.0)
        A, B = synth.uniform_patch(n, patch, rng), synth.uniform_patch(m, patch, rng)
        if where == "sorted":  # neighbours in the sky 32 places apart in the catalogue
            o = np.argsort(A[0])
            o = np.concatenate([o[k::32] for k in range(32)])
            A = (A[0][o], A[1][o])
    for e in (LOG, EVEN):
        assert pc.pc_count(dev(A), e).tolist() == oracle.count(A, e).tolist()
        assert pc.pc_count(A, e, B=dev(B), auto=False).tolist() == oracle.count(A, e, B=B, auto=False).tolist()
    r = (n // 3, n - n // 5)
    assert pc.pc_count_ex(dev(A), LOG, rows=r).tolist() == oracle.count(A, LOG, rows=r).tolist()


@pytest.mark.parametrize("jobs", [3, 40])
def test_batches_on_both_sides(jobs):
    """Forty jobs of 1400 x 600 pairs pass the line together, three do not;
    more descriptors than go as arguments in the larger one."""
    rng = np.random.default_rng(jobs)
    patch = synth.centred_patch(9.0)
    R = synth.uniform_patch(1400, patch, rng)
    D = [synth.uniform_patch(600 + k, patch, rng) for k in range(jobs)]
    dR = dev(R)
    got = pc.pc_count_batch([{"A": dev(d), "B": dR, "edges": LOG if k % 2 else EVEN, "auto": False}
                             for k, d in enumerate(D)])
    for k, d in enumerate(D):
        assert got[k].tolist() == oracle.count(d, LOG if k % 2 else EVEN, B=R, auto=False).tolist()
    h = pc.pc_catalog_upload(dR)
    try:
        assert pc.pc_count_h(h, EVEN).tolist() == oracle.count(R, EVEN).tolist()
    finally:
        pc.pc_catalog_release(h)
