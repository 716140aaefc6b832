"""The spatial ordering of a launch's catalogues on shapes where its key grid
degenerates or its blocks end: counts must equal the oracle's whatever order
the points are put in."""
import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(c):
    return tuple(torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in c)


def shape(kind, n, rng):
    if kind == "identical":                      # one cell of one face
        return np.full(n, 123.25), np.full(n, -7.5)
    if kind == "meridian":                       # a line across three faces
        return np.full(n, 10.0), np.linspace(-90.0, 90.0, n) if n > 1 else np.zeros(1)
    if kind == "strip":                          # 80 x 0.01 degrees across a face edge
        return 5.0 + 80.0 * rng.random(n), 0.01 * rng.random(n)
    if kind == "two_patches":                    # opposite faces, very different extents
        a = synth.uniform_patch(n - n // 3, synth.centred_patch(0.05), rng)
        b = synth.uniform_patch(n // 3, synth.centred_patch(40.0, ra0=160.0), rng)
        return tuple(np.concatenate([x, y]) for x, y in zip(a, b))
    return synth.uniform_patch(n, synth.FULL_SKY, rng)


@pytest.mark.parametrize("kind", ["identical", "meridian", "strip", "two_patches", "sky"])
def test_shapes_and_block_edges_match_the_oracle(kind):
    """1 .. 4097 points: edges of tiles (256), of ordering blocks (1024 points)
    and of scan blocks (4096 counters, 4 a point); DD and DR in one launch."""
    rng = np.random.default_rng(91)
    e = np.array([0.0, 0.004, 0.03, 0.5, 3.0, 20.0, 90.0, 170.0])
    for n in (1, 2, 63, 255, 257, 1023, 1025, 4097):
        A, B = shape(kind, n, rng), synth.uniform_patch(n % 700 + 3, synth.FULL_SKY, rng)
        dd, dr = pc.pc_count_batch([{"A": dev(A), "edges": e}, {"A": dev(A), "B": dev(B), "edges": e, "auto": False}])
        assert dd.tolist() == oracle.count(A, e).tolist(), n
        assert dr.tolist() == oracle.count(A, e, B=B, auto=False).tolist(), n


@pytest.mark.parametrize("mode", [pc.PC_MIXED, pc.PC_MIXED | pc.PC_NO_PRUNE, pc.PC_FP64_PLAIN,
                                  pc.PC_MIXED | pc.PC_MATRIX_CORES])
def test_many_views_in_one_launch_match_the_oracle(mode):
    """Forty catalogues of 0 to 600 points (host and device), each with its own
    key grid, against a shared one, whole and as row ranges: every ordered copy
    gets exactly its own points."""
    rng = np.random.default_rng(92)
    e = synth.log_edges(0.05, 30.0, 9)
    R = synth.uniform_patch(900, synth.centred_patch(25.0), rng)
    Rd = dev(R)
    jobs, want = [], []
    for k in range(40):
        n = int(rng.integers(0, 600)) if k else 0
        A = synth.uniform_patch(n, synth.centred_patch(float(rng.uniform(0.1, 25.0))), rng)
        A = tuple(np.asarray(x, dtype=np.float64) for x in A)
        rows = (n // 4, n - n // 5) if k % 3 == 0 else (0, n)
        Ad = dev(A) if k % 2 else A
        jobs.append({"A": Ad, "edges": e, "rows": rows})
        want.append(oracle.count(A, e, rows=rows))
        jobs.append({"A": Ad, "B": Rd, "edges": e, "auto": False, "rows": rows})
        want.append(oracle.count(A, e, B=R, auto=False, rows=rows))
    for q, (g, w) in enumerate(zip(pc.pc_count_batch(jobs, mode=mode), want)):
        assert g.tolist() == w.tolist(), (q, jobs[q]["rows"])
