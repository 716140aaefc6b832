"""pc_debug_last_pruning's item figures of the block kernel: a tile pair whose
open blocks lie in the last columns of blocks only is one item with open blocks,
whether it is taken in sixteenths, in quarters or whole."""
import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("jobs", [1, 700, 4200])
def test_items_with_open_blocks(jobs):
    rng = np.random.default_rng(8)
    A = 10.0 + 1e-3 * rng.random(512), 1e-3 * rng.random(512)
    r = np.concatenate([1.0 + 0.01 * rng.random(256), 2.9 + 0.2 * rng.random(256)])   # one bin; across an edge
    B = 10.0 + r, 1e-3 * rng.random(512)
    e = np.array([0.5, 2.0, 3.0, 10.0])
    a, b = (tuple(torch.from_numpy(x).cuda() for x in c) for c in (A, B))
    got = pc.pc_count_batch([{"A": a, "B": b, "edges": e, "auto": False}] * jobs)
    p = pc.pc_debug_last_pruning()
    assert (p["survivors"], p["split_items"], p["few_items"], p["gram_items"]) == (jobs,) * 4, p
    want = oracle.count(A, e, B=B, auto=False).tolist()
    assert all(g.tolist() == want for g in got)


def test_pairs_of_the_matrix_cores():
    """Chords of tiles far apart come from the product, some of a tile with itself
    from differences, those of binary64 launches from neither."""
    rng = np.random.default_rng(9)
    A = 10.0 + rng.random(700), rng.random(700)
    B = 60.0 + rng.random(900), rng.random(900)
    a, b = (tuple(torch.from_numpy(x).cuda() for x in c) for c in (A, B))
    e = np.array([0.01, 0.1, 49.8, 50.0, 50.2])
    pc.pc_count(a, e, B=b, auto=False)
    p, n = pc.pc_debug_last_paths(), pc.pc_debug_last_pruning()["pairs_computed"]
    assert n > 0 and p["mfma"] == n and p["gram"] == 0
    pc.pc_count(a, e)
    p, n = pc.pc_debug_last_paths(), pc.pc_debug_last_pruning()["pairs_computed"]
    assert 0 <= p["mfma"] < n and p["gram"] == 0
    pc.pc_count_ex(a, e, mode=pc.PC_FP64_PLAIN)
    p = pc.pc_debug_last_paths()
    assert p["mfma"] == 0 and p["gram"] == 0
