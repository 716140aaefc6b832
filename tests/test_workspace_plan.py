"""The device workspace a launch plans for itself, on the host."""
import pytest

import paper_1208_3658_amd as pc
import synth


def test_the_last_piece_holds_the_descriptors_whole_words():
    """The descriptors are the workspace's last piece, and a launch writes them in
    16-byte words: a launch of two sources and three segments (a row range's
    triangle and rectangle, and its cross count) has 8 bytes in the last word,
    and the workspace holds all of it."""
    needs = [p["need_bytes"] for p in pc.pc_debug_request_parts(40_000, 30_000, 21, False, 3e8)]
    needs += [p["need_bytes"] for p in pc.pc_debug_request_parts(40_000, 30_000, 21, True, 3e8)]
    assert len(needs) > 6
    assert all(n % 16 == 0 for n in needs), needs


MODES = {"mixed": pc.PC_MIXED, "binary64": pc.PC_FP64_PLAIN, "matrix_cores": pc.PC_MIXED | pc.PC_MATRIX_CORES,
         "no_prune": pc.PC_MIXED | pc.PC_NO_PRUNE}


@pytest.mark.parametrize("mode", sorted(MODES))
@pytest.mark.parametrize("views,n", [(540, 5000), (2600, 1000), (60, 30_000), (1, 900_000)])
def test_batches_that_fitted_the_fixed_area_fit(views, n, mode):
    """The workspace of a batch: 64 bytes a point of its ordered copies, 32 of
    the converted ones, the tile bounds, and 16 per pair of 256-point tiles.
    Batches that fit the fixed area with one scratch for the largest catalogue
    still do, the ordering taking several rounds where its counters do not fit."""
    e = synth.log_edges(0.02, 5.0, 20)
    need = pc.pc_debug_static_plan([n] * views, e, MODES[mode])
    assert need <= pc.PC_STATIC_SCRATCH_BYTES, need
    # and with the area cut to the ordered and converted copies, the bounds and the survivors
    tiles = -(-n // 256)
    least = views * ((128 if "matrix" in mode else 112) * n + 256 * tiles + 8 * tiles * (tiles + 1) + 2048) + (1 << 20)
    assert pc.pc_debug_static_plan([n] * views, e, MODES[mode], least) <= least


def test_dense_edge_sets_fit_by_leaving_their_chord_table():
    """A chord table of 1023 even bins takes 180 KB; an area that holds the batch
    without it is enough."""
    e = synth.linear_edges(0.0, 10.0, 1023)
    whole = pc.pc_debug_static_plan([5000], e, pc.PC_MIXED, 1 << 30)
    assert pc.pc_debug_static_plan([5000], e, pc.PC_MIXED, whole - 150_000) <= whole - 150_000
    assert pc.pc_debug_static_plan([5000], e, pc.PC_MIXED, whole - 400_000) > whole - 400_000
