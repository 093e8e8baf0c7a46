"""The 2D adjoint's set launches (P <= 3: all corner classes in one launch, or above
150000 corners at P = 3 in two, of which the second holds those with an order 3) against the launches per
class of P = 4, with the same forced orders of at most 3.  Every corner runs the
same arithmetic in both, so only the gather's summation order and the compiler's
contraction differ: at most 4 P^2 = 64 contributions of comparable size per cell
and component, 64 * 2^-53 * 4 (cancellation within a corner) < 1e-13 relative to
the largest value; bound 1e-12.
"""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

BOUND = 1e-12


def state(nx, ny):
    X, Y = np.meshgrid((np.arange(nx) + 0.5) / nx, (np.arange(ny) + 0.5) / ny, indexing="xy")
    rho = 1.0 + 0.1 * np.sin(2 * np.pi * X) * np.cos(2 * np.pi * Y)
    v, w = 0.3 + 0.05 * np.sin(2 * np.pi * Y), -0.2 + 0.05 * np.cos(2 * np.pi * X)
    return workloads.euler2d_conserved(rho, v, w, 1.0 + 0.05 * np.sin(2 * np.pi * (X + Y)))


def adjoint(acat, P, bc, u, ub, ordx, ordy):
    ny, nx = u.shape[1:]
    pg = acat.Problem(dim=2, nvar=4, nx=nx, ny=ny, flux="euler", P=P, bc=bc, dx=1.0 / nx, dy=1.0 / ny)
    dec = acat.Decisions(pg)
    for t, o in ((dec.order_x, ordx), (dec.order_y, ordy)):
        t.copy_(torch.from_numpy(o))
    for t in (dec.psi1_x, dec.psi1_y):
        t.fill_(0.6)
    for t in (dec.alpha_x, dec.alpha_y):
        t.fill_(2.0)
    return acat.step_adjoint(pg, u, 0.1 / max(nx, ny), dec, ub).cpu().numpy()


@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
@pytest.mark.parametrize("P,kind", [(1, "all"), (2, "all"), (2, "rare"), (3, "all"), (3, "rare"), (3, "top"),
                                    (3, "low")])
def test_sets_equal_the_launches_per_class(acat, P, kind, bc):
    # corners below, at and above one round of every class (256, 64, 28, 20, 16, 10, 7, ...)
    # and more rounds than resident blocks; "rare": one interface row and column off the
    # common order; "top" / "low": the second / first set only
    for nx, ny in ((8, 8), (9, 8), (10, 26), (65, 130), (150, 140)) + ((401, 380),) * (P == 3):
        rng = np.random.default_rng(nx * ny + P)
        ext = 0 if bc == "periodic" else 1
        sx, sy = (ny, nx + ext), (ny + ext, nx)
        if kind == "all":
            ordx, ordy = (rng.integers(1, P + 1, s).astype(np.int8) for s in (sx, sy))
        elif kind == "rare":
            ordx, ordy = (np.full(s, P, np.int8) for s in (sx, sy))
            ordx[ny // 2, 1] = 1
            ordy[1, nx // 2] = P - 1
        else:
            ordx, ordy = (np.full(s, P if kind == "top" else P - 1, np.int8) for s in (sx, sy))
        u = torch.from_numpy(np.ascontiguousarray(state(nx, ny))).cuda()
        ub = torch.from_numpy(rng.standard_normal((4, ny, nx))).cuda()
        got = adjoint(acat, P, bc, u, ub, ordx, ordy)
        want = adjoint(acat, 4, bc, u, ub, ordx, ordy)
        err = np.abs(got - want).max() / np.abs(want).max()
        print(f"P={P} {kind} {bc} {nx}x{ny}: {err:.2e}", flush=True)
        assert np.isfinite(got).all() and err <= BOUND, (nx, ny)
