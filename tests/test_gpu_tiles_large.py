"""1D steps of many tiles of several rounds each, against sides that are not the tile
kernel: the oracle (a whole step at 40009 cells, windows of 1500 at 300007), for orders
up to 8 a batch of the one problem by passes, and for the time step the separate
reduction; recorded and unrecorded, bit for bit.  Non-finite states against the passes
too."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_helpers import both_problems

pytestmark = pytest.mark.gpu

M = 1500


def state(flux, n):
    rng = np.random.default_rng(n)
    x = (np.arange(n) + 0.5) / n
    noise = 1e-3 * rng.standard_normal(n) * (((x > 0.3) & (x < 0.45)) | ((x > 0.8) & (x < 0.82)))
    ripple = 0.02 * np.sin(2 * np.pi * np.arange(n) / 9.3) * (np.abs(x - 0.55) < 0.03)
    if flux != "euler":
        return (0.6 + np.sin(2 * np.pi * x) + 0.5 * (x > 0.7) + noise + ripple)[None].copy()
    rho = 1.0 + 0.3 * np.sin(2 * np.pi * x) + 0.5 * (x > 0.6) + noise + ripple
    return workloads.euler1d_conserved(rho, 0.2 * np.cos(2 * np.pi * x) + noise, 1.0 + 0.2 * np.sin(4 * np.pi * x) +
                                       1.0 * (x < 0.2))


def by_passes(acat, prob, u, dt):
    batch = acat.Batch([prob.nx], [prob.P], [prob.bc], [prob.dx], flux=prob.flux, nvar=prob.nvar)
    batch.set_launch({p: (4, 0) for p in batch.orders})
    return batch.step(u, dt)


@pytest.mark.parametrize("P", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
@pytest.mark.parametrize("flux", ["euler", "burgers"])
def test_large_steps_equal_the_oracle(acat, flux, bc, P):
    for n in (40009, 300007):
        u = np.ascontiguousarray(state(flux, n))
        po, pg = both_problems(1, u.shape[0], n, flux, P, bc, 1.0 / n)
        ug, dec = torch.from_numpy(u).cuda(), acat.Decisions(pg)
        dt, want_dt = (torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2))
        acat.cfl_dt(pg, acat.max_wave_speed(pg, ug), 0.5, want_dt)
        a = acat.step_cfl(pg, ug, 0.5, dt)
        assert torch.equal(dt, want_dt), n
        recorded = acat.step_cfl(pg, ug, 0.5, dt, dec=dec)
        assert torch.equal(recorded, a) and torch.equal(dt, want_dt), n
        if P <= 4:
            assert torch.equal(by_passes(acat, pg, ug, dt), a), n
        got, h = a.cpu().numpy(), float(dt.item())
        if n < 100000:
            r = oracle.step1d(po, u, h)
            assert np.array_equal(got, r["u"]), n
            for t, name in ((dec.order_x, "order"), (dec.psi1_x, "psi1"), (dec.alpha_x, "alpha")):
                assert np.array_equal(t.cpu().numpy(), r[name]), (n, name)
            continue
        edge = 2 * P + 2
        wo, _ = both_problems(1, u.shape[0], M, flux, P, "transmissive", 1.0 / n)
        starts = [0, n - M] + [int(c * n) - M // 2 for c in (0.2, 0.3, 0.45, 0.55, 0.6, 0.8, 0.93)]
        for s in starts + ([-M // 2] if bc == "periodic" else []):
            cells = np.arange(s, s + M) % n
            w = oracle.step1d(wo, np.ascontiguousarray(u[:, cells]), h)["u"]
            lo = 0 if bc == "transmissive" and s == 0 else edge
            hi = M if bc == "transmissive" and s == n - M else M - edge
            assert np.array_equal(got[:, cells[lo:hi]], w[:, lo:hi]), s


def test_non_finite_states_equal_the_passes(acat):
    n = 1000
    u = torch.from_numpy(np.ascontiguousarray(state("euler", n))).cuda()
    u[0, 500], u[2, 700], u[1, 3] = float("nan"), float("inf"), float("-inf")
    prob = acat.Problem(dim=1, nvar=3, nx=n, flux="euler", P=4, bc="transmissive", dx=1.0 / n)
    dt = torch.full((1,), 1e-4, dtype=torch.float64, device="cuda")
    acat.device_status()
    a = acat.step(prob, u, dt)
    assert acat.device_status() & acat.DEV_NONFINITE
    b = by_passes(acat, prob, u, dt)
    assert torch.equal(torch.isfinite(a), torch.isfinite(b))
    keep = torch.isfinite(a)
    assert torch.equal(a[keep], b[keep]) and not keep.all() and int(keep.sum()) > 2 * n
