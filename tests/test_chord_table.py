"""The block kernel's chord table on the host: which edge sets have one, and that
a chord known to within an eighth of its cell is binned right by its cell's edge
alone wherever it is farther than that from the edge."""
import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc
import synth

SETS = {f"even_{k}": synth.linear_edges(0.0, 10.0, k) for k in (4, 30, 60, 100, 200, 500, 1000, 1023)}
SETS.update({f"log_{k}": synth.log_edges(0.01, 20.0, k) for k in (12, 40, 150, 254, 300, 400, 500, 700, 1023)})
SETS["wide_1023"] = synth.log_edges(1e-3, 170.0, 1023)
SETS["even_from_1"] = synth.linear_edges(1.0, 10.0, 300)
SETS.update({f"even_{k}_to_{hi}": synth.linear_edges(0.0, float(hi), k) for k, hi in ((100, 180), (179, 180), (400, 178), (1023, 170))})


@pytest.mark.parametrize("name", sorted(SETS))
def test_chords_are_placed_by_their_cell(name):
    e64 = oracle.chord2_edges(SETS[name])
    shift, key0, edge, row = pc.pc_debug_chord_table(SETS[name])
    assert edge.size > 0, "no chord table"
    rng = np.random.default_rng(7)
    near = e64[e64 > 0][:, None] * (1.0 + np.concatenate([-10.0 ** np.arange(-8, 0.0), 10.0 ** np.arange(-8, 0.0)]))
    first = e64[e64 > 0][0]
    c = np.concatenate([near.ravel(), np.exp(rng.uniform(np.log(first / 4), np.log(min(4.0, e64[-1] * 2)), 200_000))])
    q = c * 2.0 ** (shift - 26)
    for d in (-0.5, -0.1, 0.0, 0.3, 0.5):        # the chord as known, up to q / 2 off
        x = (c + d * q).astype(np.float32)
        cell = np.clip((x.view(np.uint32) >> shift).astype(np.int64) - key0, 0, edge.size - 1)
        at = row[cell] + (edge[cell] < x)
        clear = np.abs(edge[cell].astype(np.float64) - x) > 0.5 * q * (1 + 1e-6) + x * 2.0 ** -22
        want = np.searchsorted(e64, c, side="right")
        assert np.array_equal(at[clear], want[clear]), (name, d)
        assert clear.mean() > 0.3
