"""The device workspace a launch plans for itself, on the host."""
import paper_1208_3658_amd as pc


def test_the_last_piece_holds_the_descriptors_whole_words():
    """The descriptors are the workspace's last piece, and a launch writes them in
    16-byte words: a launch of two sources and three segments (a row range's
    triangle and rectangle, and its cross count) has 8 bytes in the last word,
    and the workspace holds all of it."""
    needs = [p["need_bytes"] for p in pc.pc_debug_request_parts(40_000, 30_000, 21, False, 3e8)]
    needs += [p["need_bytes"] for p in pc.pc_debug_request_parts(40_000, 30_000, 21, True, 3e8)]
    assert len(needs) > 6
    assert all(n % 16 == 0 for n in needs), needs
