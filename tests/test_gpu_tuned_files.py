"""Tuning files written before the block kernel: their columns and chunk belong to
the vector kernel, and the block kernel keeps its own."""
import json

import numpy as np
import pytest

import oracle
import paper_1208_3658_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,same", [(None, True), ("vector", True), ("blocks", False)])
def test_columns_of_the_other_kernel_are_not_taken(tmp_path, kernel, same):
    rng = np.random.default_rng(41)
    A = synth.uniform_patch(9001, synth.centred_patch(10.0), rng)
    a, e = tuple(torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in A), synth.log_edges(0.01, 8.0, 20)
    want = oracle.count(A, e).tolist()
    file = tmp_path / "tune.jsonl"
    _, cfg = pc.pc_autotune([{"A": a, "edges": e}])
    assert cfg["kernel"] == ("blocks" if cfg["tile"] == 256 and not cfg["matrix_cores"] else "vector")
    entry = {k: v for k, v in cfg.items() if k != "candidates"}
    try:
        entry.update(tile=256, cols=4, chunk=8, matrix_cores=0)
        entry.pop("kernel")
        if kernel:
            entry["kernel"] = kernel
        file.write_text(json.dumps(entry) + "\n")
        pc.pc_autotune_load(file)
        assert pc.pc_count_ex(a, e).tolist() == want
        lds = pc.pc_debug_last_launch()["lds_bytes"]
        assert pc.pc_count_ex(a, e, mode=pc.PC_MIXED | pc.PC_TUNED).tolist() == want
        assert (pc.pc_debug_last_launch()["lds_bytes"] == lds) == same
    finally:
        entry.update(cols=0, chunk=4, kernel="blocks")
        file.write_text(json.dumps(entry) + "\n")
        pc.pc_autotune_load(file)
