"""The 2D adjoint of grids above the line from which the square class (P, P) has a
launch of its own, against the launches per class of P = 4 with the same forced
orders, for Euler and advection and both boundaries; and which launches ran on
either side of the line.  Bound as for the sets of small grids: the same arithmetic per
corner, up to 64 contributions per cell summed in another order and contracted
differently, 64 * 2^-53 * 4 < 1e-13 relative to the largest value; 1e-12."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

# corners of the line and launches above it
LINE = {("euler", 2): (300000, 2), ("euler", 3): (150000, 3), ("advection", 2): (120000, 2),
        ("advection", 3): (100000, 2)}


def state(flux, nx, ny):
    X, Y = np.meshgrid((np.arange(nx) + 0.5) / nx, (np.arange(ny) + 0.5) / ny, indexing="xy")
    if flux == "advection":
        return (1.0 + 0.3 * np.sin(2 * np.pi * X) * np.cos(4 * np.pi * Y))[None]
    return workloads.euler2d_conserved(1.0 + 0.1 * np.sin(2 * np.pi * X) * np.cos(2 * np.pi * Y),
                                       0.3 + 0.05 * np.sin(2 * np.pi * Y), -0.2 + 0.05 * np.cos(2 * np.pi * X),
                                       1.0 + 0.05 * np.sin(2 * np.pi * (X + Y)))


def adjoint(acat, flux, P, bc, u, ub, orders):
    ny, nx = u.shape[1:]
    pg = acat.Problem(dim=2, nvar=u.shape[0], nx=nx, ny=ny, flux=flux, P=P, bc=bc, dx=1.0 / nx, dy=1.0 / ny, ax=0.8,
                      ay=-0.6)
    dec = acat.Decisions(pg)
    for t, o in zip((dec.order_x, dec.order_y), orders):
        t.copy_(torch.from_numpy(o))
    for t, v in ((dec.psi1_x, 0.6), (dec.psi1_y, 0.6), (dec.alpha_x, 2.0), (dec.alpha_y, 2.0)):
        t.fill_(v)
    acat.profile(True)
    out = acat.step_adjoint(pg, u, 0.1 / max(nx, ny), dec, ub).cpu().numpy()
    ran = acat.profile_read()
    acat.profile(False)
    return out, {k for k in ran if k.startswith("adjoint2d_")}


@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
@pytest.mark.parametrize("flux,P", sorted(LINE))
def test_square_class_alone_on_large_grids(acat, flux, P, bc):
    ext = 0 if bc == "periodic" else 1
    nx = 400 - ext
    line, launches = LINE[flux, P]
    for above in (False, True):
        ny = line // 400 + above - ext
        rng = np.random.default_rng(P + 10 * above)
        sx, sy = (ny, nx + ext), (ny + ext, nx)
        # mostly the highest order, as in smooth flow, a quarter drawn from all
        ordx, ordy = (np.where(rng.random(s) < 0.75, P, rng.integers(1, P + 1, s)).astype(np.int8) for s in (sx, sy))
        u = torch.from_numpy(np.ascontiguousarray(state(flux, nx, ny))).cuda()
        ub = torch.from_numpy(rng.standard_normal(tuple(u.shape))).cuda()
        got, ran = adjoint(acat, flux, P, bc, u, ub, (ordx, ordy))
        want, _ = adjoint(acat, flux, 4, bc, u, ub, (ordx, ordy))
        assert (f"adjoint2d_q{P}{P}" in ran) == above and len(ran) == (launches if above else 1), ran
        err = np.abs(got - want).max() / np.abs(want).max()
        print(f"{flux} P={P} {bc} {nx}x{ny}: {err:.2e}", flush=True)
        assert np.isfinite(got).all() and err <= 1e-12
