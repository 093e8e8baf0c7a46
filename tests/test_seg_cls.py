"""AdjointRun.seg_cls: the class counts of the steps that the first buffer set holds,
read from their workspaces' headers (host buffers here: nothing is launched)."""
import torch

import paper_2007_01416_amd as acat


def test_counts_of_the_first_buffer_set():
    prob = acat.Problem(dim=1, nvar=1, nx=64, flux="burgers", P=3, dx=1.0 / 64)
    run = acat.AdjointRun(prob, 0.4, nsteps=7, checkpoint_every=3, device="cpu", overlap=False, graphs=False)
    for j, w in enumerate(run.seg_ws):
        w[:64].view(torch.int32).copy_(torch.arange(16, dtype=torch.int32) + 100 * j)
    c = run.seg_cls
    assert c.dtype == torch.int32 and tuple(c.shape) == (3, 16)
    assert torch.equal(c, torch.arange(16, dtype=torch.int32) + 100 * torch.arange(3, dtype=torch.int32)[:, None])
