"""The 1D adjoint of large problems, whose orders go in several launches, whose tiles
take several rounds and whose scalar order 6 is shared out in stretches, against the
adjoint of overlapping windows of 4000 cells with the same decisions (one launch of few
tiles, which smaller tests compare with the oracle's dense adjoint): away from a
window's cut the adjoint of a cell depends on nothing outside it.  Same products,
contracted by the compiler in another kernel: 1e-11 of the largest value, as there.
Sizes on both sides of each line."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

M = 4000    # cells per window


def state(n, flux):
    rng = np.random.default_rng(n)
    x = (np.arange(n) + 0.5) / n
    # rough where sin > 0.4, about a third of the grid, in three stretches: order 1 there, high between
    noise = 1e-3 * rng.standard_normal(n) * (np.sin(6 * np.pi * x) > 0.4)
    # and a wave short enough that the higher orders give way to lower ones
    ripple = 0.05 * np.sin(2 * np.pi * np.arange(n) / 9.3) * (np.abs(x - 0.46) < 0.02)
    if flux != "euler":
        return (0.3 + np.sin(2 * np.pi * x) + (x > 0.7) + noise + ripple)[None]
    rho = 1 + 0.3 * np.sin(2 * np.pi * x) + 0.5 * (x > 0.6) + noise + ripple
    v, p = 0.2 * np.cos(2 * np.pi * x), 1 + 0.8 * (x < 0.25)
    return np.stack([rho, rho * v, p / 0.4 + 0.5 * rho * v * v])


@pytest.mark.parametrize("flux,P,n", [("euler", 3, 100003), ("euler", 4, 149990), ("euler", 4, 150001),
                                      ("euler", 5, 50001), ("euler", 6, 49990), ("euler", 6, 50001),
                                      ("burgers", 4, 150001), ("burgers", 5, 125001), ("burgers", 6, 124990),
                                      ("burgers", 6, 125001), ("advection", 6, 400003)])
@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
def test_large_adjoint_equals_its_windows(acat, flux, P, n, bc):
    per = bc == "periodic"
    u = torch.from_numpy(np.ascontiguousarray(state(n, flux))).cuda()
    nv = u.shape[0]
    prob = acat.Problem(dim=1, nvar=nv, nx=n, flux=flux, P=P, bc=bc, dx=1.0 / n, ax=-0.7)
    ws, dec, dt = acat.workspace(prob), acat.Decisions(prob), torch.zeros(1, dtype=torch.float64, device="cuda")
    acat.step_cfl(prob, u, 0.4, dt, ws=ws, dec=dec)
    seen = torch.bincount(dec.order_x.to(torch.int64), minlength=P + 1)
    assert seen[1] > 1000 and seen[P] > 1000 and seen[2:P].sum() > 100, seen.tolist()
    ub = torch.from_numpy(np.random.default_rng(P).standard_normal((nv, n))).cuda()
    got = acat.step_adjoint_lists(prob, u, dt, dec, ub, ws)
    assert torch.equal(acat.step_adjoint(prob, u, dt, dec, ub), got)
    assert torch.equal(acat.step_adjoint_lists(prob, u, dt, dec, ub, ws), got)
    edge = 2 * P + 2
    sub = acat.Problem(dim=1, nvar=nv, nx=M, flux=flux, P=P, bc="transmissive", dx=1.0 / n, ax=-0.7)
    sdec, aws = acat.Decisions(sub), acat.adjoint_workspace(sub)
    want = torch.full_like(got, float("nan"))
    starts = list(range(0, n - M, M - 2 * edge)) + [n - M]
    if per:
        starts.append(-M // 2)      # across the wrap
    for a in starts:
        cells = torch.arange(a, a + M, device="cuda") % n
        ifs = torch.arange(a - 1, a + M, device="cuda") % n if per else torch.arange(a, a + M + 1, device="cuda")
        for t, s in zip((sdec.order_x, sdec.psi1_x, sdec.alpha_x), (dec.order_x, dec.psi1_x, dec.alpha_x)):
            t.copy_(s[ifs])
        w = acat.step_adjoint(sub, u[:, cells].contiguous(), dt, sdec, ub[:, cells].contiguous(), ws=aws)
        lo = 0 if not per and a == 0 else edge
        hi = M if not per and a == n - M else M - edge
        want[:, cells[lo:hi]] = w[:, lo:hi]
    assert bool(torch.isfinite(want).all())
    err = float((got - want).abs().max() / want.abs().max())
    print(f"{flux} P={P} n={n} {bc}: {err:.2e}", flush=True)
    assert err <= 1e-11
