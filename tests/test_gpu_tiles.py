"""The 1D step by tiles (no decisions recorded) against the step that
records them, and the batched step by tiles against the one with a
launch per order class: the same operations per interface, so the same bits.
Sizes around the edges of a tile: the smallest grids, one cell more or less
than a tile and than the block that steps a whole problem, grids of several
rounds per wave and of more wave-speed blocks than partial maxima."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def data(flux, n, seed):
    rng = np.random.default_rng(seed)
    x = (np.arange(n) + 0.5) / n
    rough = 1e-3 * rng.standard_normal(n) * ((x > 0.3) & (x < 0.45))
    if flux != "euler":
        return (0.6 + np.sin(2 * np.pi * x) + 0.5 * (x > 0.7) + rough)[None].copy()
    rho = 1.0 + 0.3 * np.sin(2 * np.pi * x) + 0.5 * (x > 0.6) + rough
    v = 0.2 * np.cos(2 * np.pi * x) + rough
    p = 1.0 + 0.2 * np.sin(4 * np.pi * x) + 1.0 * (x < 0.2)
    return workloads.euler1d_conserved(rho, v, p)


def sizes(P):
    per = 4 * (64 // (2 * P))            # interfaces of one round of a block's four waves
    rmax = 256 // per
    out = {2 * max(P, 2), 2 * max(P, 2) + 1, per - 2, per - 1, per, per + 1, 4 * per - 1, 4 * per,
           per * rmax - 1, per * rmax, 254, 255, 256, 257}
    return sorted(n for n in out if n >= 2 * max(P, 2)) + [40009, 300007]


@pytest.mark.parametrize("P", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
@pytest.mark.parametrize("flux", ["euler", "burgers"])
def test_tiles_equal_passes(acat, flux, bc, P):
    import torch
    variants = (0,) if flux == "euler" else (0, acat.FLAG_PSI2_MODIFIED | acat.FLAG_PSI1_ROE)
    for n in sizes(P):
        u = torch.from_numpy(data(flux, n, n)).cuda()
        for flags in variants + ((acat.FLAG_FLO_LF, acat.FLAG_FLO_HLL) if n == 257 else ()):
            prob = acat.Problem(dim=1, nvar=u.shape[0], nx=n, flux=flux, P=P, bc=bc, dx=1.0 / n, flags=flags)
            dec = acat.Decisions(prob)
            res = []
            for d in (dec, None):
                dt, t = (torch.full((1,), v, dtype=torch.float64, device="cuda") for v in (0.0, 0.25))
                a = acat.step_cfl(prob, u, 0.5, dt, t, dec=d)
                clipped = torch.zeros_like(dt)
                b = acat.step_cfl(prob, u, 0.5, clipped, t, 0.25 + 1.25 * float(dt.item()), dec=d)
                c = acat.step(prob, u, 0.3 / n / 4, dec=d)
                res.append((a, dt, t, b, clipped, c))
            for k, (x, y) in enumerate(zip(*res)):
                assert torch.equal(x, y), (n, flags, k)


def test_tiles_carry_non_finite_states(acat):
    """NaN and infinite cells: the same cells of the result are not finite."""
    import torch
    n = 1000
    u = torch.from_numpy(data("euler", n, 3)).cuda()
    u[0, 500] = float("nan")
    u[2, 700] = float("inf")
    prob = acat.Problem(dim=1, nvar=3, nx=n, flux="euler", P=4, bc="transmissive", dx=1.0 / n)
    acat.device_status()
    a = acat.step(prob, u, 1e-4, dec=acat.Decisions(prob))
    sa = acat.device_status()
    b = acat.step(prob, u, 1e-4)
    assert sa == acat.device_status() and sa & acat.DEV_NONFINITE
    assert torch.equal(torch.isfinite(a), torch.isfinite(b))
    keep = torch.isfinite(a)
    assert torch.equal(a[keep], b[keep]) and not keep.all() and int(keep.sum()) > 2 * n


@pytest.mark.parametrize("flux", ["euler", "burgers", "advection"])
@pytest.mark.parametrize("scale", [1, 60])
def test_batch_tiles_equal_class_launches(acat, flux, scale):
    """scale 60: enough cells that a tile takes several rounds."""
    import torch
    ns = [8, 9, 31, 32, 127, 128, 129, 255, 256, 257, 513, 1000 * scale, 77 * scale, 5000 * scale, 4001 * scale]
    probs = [(n, 1 + b % 4, ("periodic", "transmissive")[(b // 2) % 2]) for b, n in enumerate(ns * 2)]
    us = [data(flux, n, b) for b, (n, _, _) in enumerate(probs)]
    batch = acat.Batch([p[0] for p in probs], [p[1] for p in probs], [p[2] for p in probs],
                       [1.0 / p[0] for p in probs], flux=flux, nvar=us[0].shape[0], ax=-0.7)
    u = torch.from_numpy(np.concatenate(us, axis=1)).cuda()
    dt0 = torch.empty(len(probs), dtype=torch.float64, device="cuda")
    batch.cfl_dt(u, 0.5, dt0)
    res = []
    for table in ({p: (4, 0) for p in batch.orders}, None):
        batch.set_launch(table)
        dt = dt0.clone()
        a = batch.step_cfl(u, dt, 0.5)
        b = batch.step(a, dt)
        check = torch.empty_like(dt)
        batch.cfl_dt(a, 0.5, check)
        res.append((a, dt, b, check))
    assert all(torch.equal(x, y) for x, y in zip(*res))
    assert torch.equal(res[1][1], res[1][3])
