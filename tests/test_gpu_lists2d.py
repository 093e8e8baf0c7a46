"""The 2D class lists in one launch (up to 1024 tiles of 16 x 16 corners) and in two:
one step on both sides of the line and at the smallest grids bit for bit against
the oracle, and the class counts against the recorded orders, for a given and
for a CFL time step, and in the adjoint that makes its own lists."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_helpers import both_problems

pytestmark = pytest.mark.gpu


def state(nx, ny):
    rng = np.random.default_rng(nx + ny)
    X, Y = np.meshgrid((np.arange(nx) + 0.5) / nx, (np.arange(ny) + 0.5) / ny, indexing="xy")
    noise = 1e-3 * rng.standard_normal((ny, nx)) * ((X > 0.6) & (X < 0.8))
    rho = 1.0 + 0.3 * np.sin(2 * np.pi * X) * np.cos(2 * np.pi * Y) + 0.4 * (X > 0.55) + noise
    return workloads.euler2d_conserved(rho, 0.2 * np.cos(2 * np.pi * Y), -0.1 + 0 * X, 1.0 + 0.8 * (Y < 0.35))


@pytest.mark.parametrize("nx,ny,P,bc", [(8, 8, 1, "periodic"), (8, 9, 4, "transmissive"), (16, 16, 2, "periodic"),
                                        (16, 16, 3, "transmissive"), (130, 67, 4, "periodic"),
                                        (512, 512, 2, "periodic"), (512, 513, 2, "periodic"),
                                        (511, 511, 1, "transmissive"), (511, 512, 1, "transmissive")])
def test_lists_in_one_launch_and_two(acat, nx, ny, P, bc):
    po, pg = both_problems(2, 4, nx, "euler", P, bc, 1.0 / nx, ny=ny, dy=1.0 / ny)
    u = np.ascontiguousarray(state(nx, ny))
    dt = oracle.dt_cfl(po, u, 0.4)
    r = oracle.step2d(po, u, dt)
    ug, ws, dec = torch.from_numpy(u).cuda(), acat.workspace(pg), acat.Decisions(pg)
    ws.fill_(255)
    assert np.array_equal(acat.step(pg, ug, dt, ws=ws, dec=dec).cpu().numpy(), r["u"])
    ox, oy = dec.order_x.cpu().numpy(), dec.order_y.cpu().numpy()
    assert np.array_equal(ox, r["ordx"]) and np.array_equal(oy, r["ordy"])
    # every corner but, transmissive, the one outside both edges, which has no flux of the grid
    total = nx * ny if bc == "periodic" else (nx + 1) * (ny + 1) - 1
    counts = ws[:4 * P * P].view(torch.int32).clone()
    assert int(counts.sum()) == total and int(counts.min()) >= 0
    ub = torch.from_numpy(np.random.default_rng(P).standard_normal(u.shape)).cuda()
    assert torch.equal(acat.step_adjoint_lists(pg, ug, dt, dec, ub, ws), acat.step_adjoint(pg, ug, dt, dec, ub))
    ws.fill_(255)
    dtd = torch.zeros(1, dtype=torch.float64, device="cuda")
    c = acat.step_cfl(pg, ug, 0.4, dtd, ws=ws)
    assert torch.equal(ws[:4 * P * P].view(torch.int32), counts)
    assert torch.equal(c, acat.step(pg, ug, dtd))
