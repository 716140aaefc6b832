"""The small tests of the ordering and of the block kernel again with the spatial
ordering forced, which their few pairs would not get, and the block kernel's ways
of binning on catalogues whose blocks the test knows: sorted here and counted in
that order, each way is shown to be reached."""
import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc
import synth
import test_gpu_blocks
import test_gpu_blocks_fp64
import test_gpu_ordering
from test_gpu_blocks import dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture
def ordered():
    pc.pc_debug_set_order(1)
    yield
    last = pc.pc_debug_last_ordered()
    pc.pc_debug_set_order(0)
    assert last


@pytest.mark.parametrize("kind", ["identical", "meridian", "strip", "two_patches", "sky"])
def test_shapes(ordered, kind):
    test_gpu_ordering.test_shapes_and_block_edges_match_the_oracle(kind)


@pytest.mark.parametrize("mode", [pc.PC_MIXED, pc.PC_FP64_PLAIN])
def test_many_views(ordered, mode):
    test_gpu_ordering.test_many_views_in_one_launch_match_the_oracle(mode)


@pytest.mark.parametrize("kind", sorted(test_gpu_blocks.EDGES))
def test_sizes(ordered, kind):
    test_gpu_blocks.test_sizes_around_groups_tiles_and_units_match_the_oracle(kind)


@pytest.mark.parametrize("kind", sorted(test_gpu_blocks.EDGES))
def test_sizes_binary64(ordered, kind):
    test_gpu_blocks_fp64.test_sizes_around_groups_tiles_and_units(kind)


def test_pairs_around_edges(ordered):
    test_gpu_blocks.test_pairs_on_and_around_edges_at_every_scale()


def test_pairs_around_edges_binary64(ordered):
    test_gpu_blocks_fp64.test_pairs_on_and_next_to_edges()


# ------------------------------------------- blocks that the test knows

def vectors(c):
    ra, dec = np.radians(c[0]), np.radians(c[1])
    return np.stack([np.cos(dec) * np.cos(ra), np.cos(dec) * np.sin(ra), np.sin(dec)], 1)


def balls(v):
    """Tiles of 512 points: centre, radius; groups of 32: centre, radius."""
    out = []
    for t in range(0, len(v), 512):
        p = v[t:t + 512]
        c = p.sum(0) / np.linalg.norm(p.sum(0))
        g = [p[k:k + 32] for k in range(0, len(p), 32)]
        out.append((c, np.sqrt(((p - c) ** 2).sum(1).max()), [x.mean(0) for x in g],
                    [np.sqrt(((x - x.mean(0)) ** 2).sum(1).max()) for x in g]))
    return out


def ways(A, B, e):
    """How many blocks of A x B the mixed block kernel bins by one or two edges, by
    three (or more, where the blocks are ragged), by the table with and without its
    clamp, and from differences."""
    e64 = oracle.chord2_edges(e)
    shift, key0, cell, _ = pc.pc_debug_chord_table(e)
    lo_t, hi_t = (float(np.array([k << shift], dtype=np.uint32).view(np.float32)[0]) for k in (key0, key0 + cell.size))
    n = dict(narrow=0, edges=0, clamped=0, inside=0, near=0)
    sa, sb = len(A[0]), len(B[0])
    for ti, (ci, ri, gi, qi) in enumerate(balls(vectors(A))):
        for tj, (cj, rj, gj, qj) in enumerate(balls(vectors(B))):
            D, R, u = np.linalg.norm(ci - cj), ri + rj, 2.0 ** -24
            E_t = u * R * (88 * D + 50 * R) + u * (14 * D * D + 2 * (D + R) ** 2)
            for k, (a, x) in enumerate(zip(gi, qi)):
                for m, (b, y) in enumerate(zip(gj, qj)):
                    d = np.linalg.norm(a - b)
                    lo, hi = max(d - x - y, 0.0) ** 2, (d + x + y) ** 2
                    edges = np.searchsorted(e64, hi, "right") - np.searchsorted(e64, lo, "right")
                    full = min(sa - 512 * ti - 32 * k, sb - 512 * tj - 32 * m) >= 32
                    if edges == 0:
                        continue
                    if lo < E_t * 2.0 ** (27 - shift):
                        n["near"] += 1
                    elif edges >= 3 and full:
                        n["inside" if lo - E_t > lo_t and hi + E_t < hi_t else "clamped"] += 1
                    else:
                        n["narrow" if edges < 3 else "edges"] += 1
    return n


def sort_cells(c, size):
    """Points in square cells of `size` degrees, row by row, back and forth."""
    y = np.floor(c[1] / size)
    x = np.floor(c[0] / size)
    o = np.lexsort((np.where(y % 2 == 0, x, -x), y))
    return c[0][o], c[1][o]


SETS = {"log": synth.log_edges(0.01, 12.0, 30), "even": synth.linear_edges(0.0, 8.0, 40),
        "few": np.array([0.4, 2.0, 7.0])}
REACHED = {"log": {"narrow", "edges", "near", "clamped"}, "even": {"narrow", "clamped", "inside", "near"},
           "few": {"narrow", "near"}}


@pytest.mark.parametrize("kind", sorted(SETS))
def test_pairs_on_and_around_edges_in_known_blocks(kind):
    """4003 and 2900 points in cells of 0.8 degrees; to 1000 points of the first
    a partner lies within 1e-12 .. 1e-5 relative of one of the edges."""
    e = SETS[kind]
    rng = np.random.default_rng(17)
    A = synth.uniform_patch(4003, synth.centred_patch(14.0), rng)
    F = synth.uniform_patch(1900, synth.centred_patch(14.0), rng)
    t = rng.choice(e[e > 0], 1000)
    eps = rng.choice([0.0, 1e-12, -1e-12, 1e-9, -1e-9, 1e-7, -1e-7, 1e-5, -1e-5], 1000)
    up = np.where(A[1][:1000] > 0, -1.0, 1.0)
    B = (np.concatenate([A[0][:1000], F[0]]), np.concatenate([A[1][:1000] + up * t * (1 + eps), F[1]]))
    A, B = sort_cells(A, 0.8), sort_cells(B, 0.8)
    n = ways(A, B, e)
    assert {k for k, v in n.items() if v >= 10} >= REACHED[kind], n
    want = oracle.count(A, e, B=B, auto=False).tolist()
    try:
        for mode, order in ((pc.PC_MIXED, -1), (pc.PC_MIXED, 1), (pc.PC_FP64_PLAIN, -1), (pc.PC_FP64_PLAIN, 1)):
            pc.pc_debug_set_order(order)
            assert pc.pc_count_ex(dev(A), e, B=dev(B), auto=False, mode=mode).tolist() == want, (mode, order)
            assert pc.pc_debug_last_ordered() == (order == 1)
    finally:
        pc.pc_debug_set_order(0)
