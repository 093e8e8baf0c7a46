"""The 2D step's flux launches: all order classes of a small grid in one launch
and of a larger one in two (the line lies at 300 x 300 corners at P = 3), and
the classification that writes every decision where they are recorded and
only those the fluxes read where they are not.  One step against the oracle on
both sides of the line; recorded and unrecorded steps against each other; all
bit for bit."""
import numpy as np
import pytest

import workloads
from gpu_helpers import both_problems
from test_gpu_parity import lockstep

pytestmark = pytest.mark.gpu


def data(nx, ny, rough=True):
    rng = np.random.default_rng(nx + ny)
    X, Y = np.meshgrid((np.arange(nx) + 0.5) / nx, (np.arange(ny) + 0.5) / ny, indexing="xy")
    noise = 1e-3 * rng.standard_normal((ny, nx)) * (((X > 0.1) & (X < 0.2)) | ((Y > 0.7) & (Y < 0.8))) * rough
    rho = 1.0 + 0.3 * np.sin(2 * np.pi * X) * np.cos(2 * np.pi * Y) + 0.4 * (X > 0.55) + noise
    v, w = 0.2 * np.cos(2 * np.pi * Y) + noise, -0.15 * np.sin(2 * np.pi * X)
    p = 1.0 + 0.2 * np.sin(2 * np.pi * (X + Y)) + 0.8 * (Y < 0.35)
    return workloads.euler2d_conserved(rho, v, w, p)


@pytest.mark.parametrize("nx,ny,bc", [(300, 300, "periodic"), (301, 300, "periodic"), (299, 299, "transmissive"),
                                      (299, 300, "transmissive")])
def test_one_launch_and_two_equal_the_oracle(acat, nx, ny, bc):
    po, pg = both_problems(2, 4, nx, "euler", 3, bc, 1.0 / nx, ny=ny, dy=1.0 / ny)
    lockstep(acat, po, pg, data(nx, ny), 0.4, 1, label=f"euler2d P=3 {bc} {nx}x{ny}")


@pytest.mark.parametrize("P", [1, 2, 3, 4])
@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
def test_unrecorded_step_equals_recorded(acat, P, bc):
    import torch
    for nx, ny in ((16, 16), (33, 47), (130, 95), (310, 305)):
        u = torch.from_numpy(np.ascontiguousarray(data(nx, ny))).cuda()
        for flags in (0, acat.FLAG_SQUARE_2D) if nx < 300 else (0,):
            prob = acat.Problem(dim=2, nvar=4, nx=nx, ny=ny, flux="euler", P=P, bc=bc, dx=1.0 / nx, dy=1.0 / ny,
                                flags=flags)
            dec = acat.Decisions(prob)
            ws = acat.workspace(prob)
            dt = torch.zeros(1, dtype=torch.float64, device="cuda")
            a = acat.step_cfl(prob, u, 0.4, dt, ws=ws, dec=dec)
            ws.fill_(255)                    # every decision left in the workspace: NaN, order -1
            dt2 = torch.zeros_like(dt)
            b = acat.step_cfl(prob, u, 0.4, dt2, ws=ws)
            assert torch.equal(a, b) and torch.equal(dt, dt2), (nx, ny, flags)
