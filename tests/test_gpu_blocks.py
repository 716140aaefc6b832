"""The block kernel (the mixed mode's pruned launches: 512-point tiles as 32 x 32
blocks, chords from matrix products) against the oracle and the other kernels,
at the sizes where its tiles, groups and work units end and in each of its ways
of binning: one or two edges, three or four, the chord table, chords from
differences, more edges than a wave has lanes, and no table at all."""
import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EDGES = {
    "one": np.array([1.3, 2.9]),                                     # blocks of one edge or two
    "zero": np.array([0.0, 0.05, 0.4, 2.0, 7.0]),                     # an edge at 0
    "log": synth.log_edges(0.01, 12.0, 30),
    "even": synth.linear_edges(0.0, 8.0, 40),                         # many edges per block: the table
    "dense": synth.log_edges(1e-3, 170.0, 1023),                      # > 64 edges inside a tile pair, no table
    "paper": synth.log_edges(0.001, 90.0, 254),
    "tight": 3.0 + 1e-7 * np.arange(12),                              # edges closer than a table cell
}


def dev(c):
    return tuple(torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in c)


@pytest.mark.parametrize("kind", sorted(EDGES))
def test_sizes_around_groups_tiles_and_units_match_the_oracle(kind):
    e = EDGES[kind]
    rng = np.random.default_rng(131)
    for n in (1, 2, 31, 32, 33, 63, 65, 511, 512, 513, 1025, 1600):
        patch = synth.centred_patch(float(rng.uniform(0.5, 14.0)))
        A = synth.uniform_patch(n, patch, rng)
        B = synth.neyman_scott(n // 20 + 1, 20, 0.03, patch, rng)
        assert pc.pc_count(dev(A), e).tolist() == oracle.count(A, e).tolist(), n
        assert pc.pc_count(dev(A), e, B=dev(B), auto=False).tolist() == oracle.count(A, e, B=B, auto=False).tolist(), n
        assert pc.pc_count(dev(B), e).tolist() == oracle.count(B, e).tolist(), n
        r = (n // 3, n - n // 4)
        assert pc.pc_count_ex(dev(A), e, rows=r).tolist() == oracle.count(A, e, rows=r).tolist(), (n, r)


@pytest.mark.parametrize("n", [700, 6000, 40000])
def test_units_of_a_sixteenth_a_quarter_and_a_whole_tile_pair(n):
    """Few survivors are cut into sixteen or four units, many are taken whole:
    equal counts from the block kernel, the vector kernel of 256-point tiles and
    the binary64 kernel, auto and cross, device, host and resident."""
    rng = np.random.default_rng(n)
    side = (n / 50.0) ** 0.5
    D = synth.neyman_scott(n // 20, 20, 0.05, synth.centred_patch(side), rng)
    R = synth.uniform_patch(n + 333, synth.centred_patch(side), rng)
    e = synth.log_edges(0.01, 0.7 * side, 25)
    jobs = [{"A": dev(D), "edges": e}, {"A": dev(D), "B": dev(R), "edges": e, "auto": False},
            {"A": R, "edges": synth.linear_edges(0.0, side, 17)}]
    got = pc.pc_count_batch(jobs)
    try:
        pc.pc_debug_set_tile(256)
        vec = pc.pc_count_batch(jobs)
    finally:
        pc.pc_debug_set_tile(0)
    f64 = pc.pc_count_batch(jobs, mode=pc.PC_FP64_PLAIN)
    for g, v, f in zip(got, vec, f64):
        assert g.tolist() == v.tolist() == f.tolist()
    h = [pc.pc_catalog_upload(dev(D)), pc.pc_catalog_upload(R)]
    try:
        assert pc.pc_count_h(h[0], e, hB=h[1], auto=False).tolist() == got[1].tolist()
        assert pc.pc_count_h(h[0], e).tolist() == got[0].tolist()
    finally:
        for x in h:
            pc.pc_catalog_release(x)


def test_pairs_on_and_around_edges_at_every_scale():
    """Pairs placed within 1e-12 .. 1e-5 relative of edges from an arcsecond to
    100 degrees, among a clustered field that makes tiles wide: every one is
    decided as the binary64 definition decides it."""
    rng = np.random.default_rng(77)
    edges = np.array([0.0003, 0.002, 0.01, 0.03, 0.1, 0.4, 1.0, 3.0, 9.0, 30.0, 100.0])
    ra, dec = [], []
    for t in edges:
        for _ in range(60):
            r0, d0 = rng.uniform(0, 40), rng.uniform(-50, 50 - min(t, 40.0))
            eps = rng.choice([0.0, 1e-12, -1e-12, 1e-9, -1e-9, 1e-7, -1e-7, 1e-5, -1e-5])
            ra += [r0, r0]
            dec += [d0, min(d0 + t * (1 + eps), 89.9)]
    F = synth.neyman_scott(60, 20, 0.02, synth.centred_patch(30.0), rng)
    A = (np.concatenate([ra, F[0]]), np.concatenate([dec, F[1]]))
    for e in (edges, synth.log_edges(0.0003, 100.0, 40), synth.log_edges(0.0003, 100.0, 300)):
        assert pc.pc_count(dev(A), e).tolist() == oracle.count(A, e).tolist()
    assert pc.pc_debug_last_rechecks() > 0
