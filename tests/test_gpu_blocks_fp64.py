"""The block kernel's binary64 instance (pruned PC_FP64_PLAIN launches) against
the oracle: sizes around its groups, tiles and work units, a few edges by
comparison, many through the chord table (in LDS and in global memory) or
without one, pairs on and next to edges, and the resident form."""
import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc
import synth
from test_gpu_blocks import EDGES, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
F64 = pc.PC_FP64_PLAIN


@pytest.mark.parametrize("kind", sorted(EDGES))
def test_sizes_around_groups_tiles_and_units(kind):
    e = EDGES[kind]
    rng = np.random.default_rng(171)
    for n in (1, 2, 31, 33, 64, 511, 513, 1100, 6100):
        patch = synth.centred_patch(float(rng.uniform(0.5, 14.0)))
        A = synth.uniform_patch(n, patch, rng)
        B = synth.neyman_scott(n // 20 + 1, 20, 0.03, patch, rng)
        assert pc.pc_count_ex(dev(A), e, mode=F64).tolist() == oracle.count(A, e).tolist(), n
        got = pc.pc_count_ex(dev(B), e, B=dev(A), auto=False, mode=F64)
        assert got.tolist() == oracle.count(B, e, B=A, auto=False).tolist(), n
        r = (n // 3, n - n // 4)
        assert pc.pc_count_ex(dev(A), e, mode=F64, rows=r).tolist() == oracle.count(A, e, rows=r).tolist(), (n, r)


def test_whole_tile_pairs_and_resident_catalogues():
    rng = np.random.default_rng(5)
    D = synth.neyman_scott(1500, 20, 0.05, synth.centred_patch(20.0), rng)
    R = synth.uniform_patch(40333, synth.centred_patch(20.0), rng)
    h = [pc.pc_catalog_upload(dev(D)), pc.pc_catalog_upload(R)]
    try:
        for e in (EDGES["log"], EDGES["even"], EDGES["paper"]):
            want = oracle.count(D, e, B=R, auto=False).tolist()
            assert pc.pc_count_ex(D, e, B=dev(R), auto=False, mode=F64).tolist() == want
            assert pc.pc_count_h(h[0], e, hB=h[1], auto=False, mode=F64).tolist() == want
            assert pc.pc_debug_last_rechecks() == 0
    finally:
        for x in h:
            pc.pc_catalog_release(x)


def test_pairs_on_and_next_to_edges():
    rng = np.random.default_rng(78)
    edges = np.array([0.0003, 0.002, 0.01, 0.03, 0.1, 0.4, 1.0, 3.0, 9.0, 30.0, 100.0])
    ra, dec = [], []
    for t in edges:
        for _ in range(60):
            r0, d0 = rng.uniform(0, 40), rng.uniform(-50, 50 - min(t, 40.0))
            eps = rng.choice([0.0, 1e-15, -1e-15, 1e-12, -1e-12, 1e-8, -1e-8, 1e-7, -1e-7, 1e-6])
            ra += [r0, r0]
            dec += [d0, min(d0 + t * (1 + eps), 89.9)]
    F = synth.neyman_scott(300, 20, 0.02, synth.centred_patch(30.0), rng)
    A = (np.concatenate([ra, F[0]]), np.concatenate([dec, F[1]]))
    for e in (edges, synth.log_edges(0.0003, 100.0, 40), synth.log_edges(0.0003, 100.0, 300)):
        assert pc.pc_count_ex(dev(A), e, mode=F64).tolist() == oracle.count(A, e).tolist()
