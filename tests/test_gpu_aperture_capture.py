"""The first aperture map of a process, made on a stream of its own while another
thread captures a graph: neither call disturbs the other.  Only the first call
uploads the filter table, hence a process of its own."""
import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CODE = """
import threading
import torch
import paper_1208_3658_amd as pc
g = torch.Generator(device="cuda").manual_seed(1)
x, y = 10.0 * torch.rand(2, 5000, generator=g, device="cuda", dtype=torch.float64)
e = 0.1 * torch.randn(2, 5000, generator=g, device="cuda", dtype=torch.float64)
cat, grid = (x.contiguous(), y.contiguous(), e[0].contiguous(), e[1].contiguous()), (0.1, 0.1, 0.2, 0.2, 50, 50)
out = {k: torch.empty(2500, dtype=t, device="cuda") for k, t in
       (("map", torch.float64), ("snr", torch.float64), ("n_in", torch.int32))}
s, a, graph, failed = torch.cuda.Stream(), torch.zeros(8, device="cuda"), torch.cuda.CUDAGraph(), []

def aperture():
    try:
        pc.pc_aperture_mass(cat, grid, 1.0, 35.0, out=out, stream=s)
    except Exception as q:
        failed.append(q)

torch.cuda.synchronize()
with torch.cuda.graph(graph, capture_error_mode="thread_local"):
    b = a + 1
    t = threading.Thread(target=aperture)
    t.start()
    t.join()
    b = b + 1
assert not failed, failed
for _ in range(3):
    graph.replay()
    torch.cuda.synchronize()
    assert b.tolist() == [2.0] * 8
again = pc.pc_aperture_mass(tuple(v.cpu().numpy() for v in cat), grid, 1.0, 35.0)
assert (out["n_in"].cpu().numpy() == again["n_in"]).all() and again["n_in"].sum() > 300000
assert (out["map"].cpu().numpy() == again["map"]).all()
"""


def test_first_map_beside_a_capture():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CODE], cwd=root, capture_output=True, text=True, timeout=90)
    assert r.returncode == 0, r.stderr[-2000:]
