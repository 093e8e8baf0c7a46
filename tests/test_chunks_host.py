"""The dynamic shares of a class list among persistent blocks, run on the CPU:
every item of the list is taken exactly once, whatever the order in which the
blocks come to their rounds."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2007_01416_amd", "csrc")


def test_every_item_taken_once(tmp_path):
    exe = str(tmp_path / "chunks_host")
    cmd = ["g++", "-std=c++20", "-O2", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-fconstexpr-ops-limit=4000000000", "-I", os.path.join(HERE, "host_kernels"), "-I", CSRC,
           "-I", os.path.join(ROOT, "include"), os.path.join(HERE, "host_kernels", "chunks_host.cpp"), "-o", exe,
           "-pthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, r.stderr[-4000:]
    bad, cases = map(int, r.stdout.split())
    assert cases > 400 and bad == 0, r.stdout
