"""The index arithmetic of the 1D adjoint at the largest sizes the library takes
(2^31 - 2 interfaces), run on the CPU under the undefined-behaviour sanitizer:
the lanes of a last tile that ends past 2^31 have no item, and the nodes of a
stencil at the end of the grid map to its cells."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2007_01416_amd", "csrc")


def test_items_and_nodes_at_the_largest_sizes(tmp_path):
    exe = str(tmp_path / "tile_items_host")
    cmd = ["g++", "-std=c++20", "-O2", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
           "-fconstexpr-ops-limit=4000000000", "-I", os.path.join(HERE, "host_kernels"), "-I", CSRC,
           "-I", os.path.join(ROOT, "include"), os.path.join(HERE, "host_kernels", "tile_items_host.cpp"), "-o", exe,
           "-pthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    bad, seen = map(int, r.stdout.split())
    assert seen > 40000 and bad == 0, r.stdout
