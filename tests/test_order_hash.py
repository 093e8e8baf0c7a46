"""The order checksums of several steps at once equal those of each step alone:
sum over positions i of order[i] ((i mod 8191) + 1) in whole numbers, axes
combined by h_x 1000003 + h_y; for any number of steps held per chunk."""
import numpy as np
import pytest
import torch

import paper_2007_01416_amd as acat
from paper_2007_01416_amd import runner


@pytest.mark.parametrize("dim,nx,ny", [(1, 17, 1), (1, 20011, 1), (2, 100, 95), (2, 16, 18)])
@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
@pytest.mark.parametrize("steps,chunk", [(1, 1 << 23), (5, 1 << 23), (5, 1), (7, 3)])
def test_hashes_of_a_segment_equal_each_steps(monkeypatch, dim, nx, ny, bc, steps, chunk):
    prob = acat.Problem(dim=dim, nvar=4 if dim == 2 else 3, nx=nx, ny=ny, flux="euler", P=3, bc=bc, dx=1.0 / nx,
                        dy=1.0 / ny)
    rng = np.random.default_rng(nx)
    decs, want = [], []
    for _ in range(steps):
        d = acat.Decisions(prob, device="cpu")
        h = None
        for t in (d.order_x, d.order_y):
            if t is None:
                continue
            o = rng.integers(-1, 7, tuple(t.shape)).astype(np.int8)
            t.copy_(torch.from_numpy(o))
            v = o.reshape(-1).astype(np.int64)
            s = int((v * (np.arange(1, v.size + 1) % 8191 + 1)).sum())
            h = s if h is None else h * 1000003 + s
        decs.append(d)
        want.append((h + 2 ** 63) % 2 ** 64 - 2 ** 63)
    w = runner._hash_weights(decs[0])
    monkeypatch.setattr(runner, "HASH_CHUNK", chunk if chunk > 3 else chunk * w.numel())
    out = torch.zeros(steps + 2, dtype=torch.int64)
    runner._order_hashes(decs, w, out[1:steps + 1])
    assert out.tolist() == [0] + want + [0]
