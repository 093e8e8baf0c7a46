"""The tiles of a batch in launch order: every cell of every problem once, the slots
of a problem side by side, the highest order first and, within an order, no tile
longer than one before it (so that no XCD gets all the long ones)."""
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("tiles") / "batch_tiles_host")
    cmd = ["g++", "-std=c++20", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-fconstexpr-ops-limit=4000000000", "-I", os.path.join(HERE, "host_kernels"), "-I",
           os.path.join(ROOT, "paper_2007_01416_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
           os.path.join(HERE, "host_kernels", "batch_tiles_host.cpp"), "-o", out, "-pthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


T = {1: 255, 2: 255, 3: 239, 4: 63}


@pytest.mark.parametrize("ns", [[256] * 40, [8, 9, 62, 63, 64, 126, 127, 238, 239, 240, 254, 255, 256, 510, 511, 5000] * 4,
                                [8], list(np.random.default_rng(1).integers(8, 2000, 300))])
def test_tiles_of_a_batch(exe, ns):
    ps = [1 + (7 * b // 3) % 4 for b in range(len(ns))]
    text = " ".join([str(len(ns))] + [f"{n} {p}" for n, p in zip(ns, ps)] + [str(T[p]) for p in (1, 2, 3, 4)])
    r = subprocess.run([exe], input=text, capture_output=True, text=True,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, r.stderr[-4000:]
    rows = [list(map(int, line.split())) for line in r.stdout.splitlines()]
    tiles, slots = rows[:-len(ns)], rows[-len(ns):]
    seen = [np.zeros(n, dtype=int) for n in ns]
    of_slot, last = {}, (5, 0)
    for b, c0, t, slot in tiles:
        assert t == T[ps[b]]
        cells = seen[b][c0:c0 + t]
        cells += 1
        assert ps[b] < last[0] or ps[b] == last[0] and len(cells) <= last[1], (b, c0)
        last = (ps[b], len(cells))
        assert slot not in of_slot
        of_slot[slot] = b
    assert all((s == 1).all() for s in seen)
    assert sorted(of_slot) == list(range(len(tiles)))
    for b, (first, count) in enumerate(slots):
        assert count == -(-ns[b] // T[ps[b]]) and all(of_slot[first + k] == b for k in range(count))


@pytest.mark.parametrize("np_, n, nvar, tiles", [
    (1, 8, 3, True), (3000, 8, 3, True), (10000, 48, 3, False), (10000, 64, 3, False), (5000, 64, 3, True), (40000, 8, 3, False),
    (40000, 100, 3, True), (3000, 8, 1, True), (10000, 16, 1, False), (10000, 48, 1, True), (40000, 64, 1, False), (300, 5000, 3, True),
    (1 << 24, 8, 3, False), (1 << 24, 100, 3, False), ((1 << 24) - 1, 100, 3, True)])
def test_many_small_problems_go_by_passes(exe, np_, n, nvar, tiles):
    """The last three: 2^24 tiles of 256 threads are more than one launch holds."""
    for p in (1, 2, 3, 4):
        r = subprocess.run([exe, "rule"], input=f"{np_} {n} {p} {nvar}", capture_output=True, text=True,
                           env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
        assert r.returncode == 0 and r.stdout.split() == [str(int(tiles))], (p, r.stderr[-2000:])
