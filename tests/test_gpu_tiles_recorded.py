"""1D steps by tiles with recorded or given decisions, and the 1D adjoint by tiles:
at the edges of tiles (smallest problem, one tile, one interface more, many
tiles), bit for bit against the oracle's step, against each other, and the class
counts against the orders.  The adjoint that reads the step's class map equals
the one that takes the recorded orders, bit for bit, and the oracle's dense
adjoint to 1e-11 of the largest value (the same products in another order)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import both_problems

pytestmark = pytest.mark.gpu

PER = {1: 128, 2: 64, 3: 40, 4: 32, 5: 24, 6: 20}    # interfaces of one round of a block


def state(n, flux):
    rng = np.random.default_rng(n)
    x = (np.arange(n) + 0.5) / n
    noise = 1e-3 * rng.standard_normal(n) * ((x > 0.3) & (x < 0.5))
    if flux == "burgers":
        return (0.3 + np.sin(2 * np.pi * x) + (x > 0.7) + noise)[None]
    rho = 1 + 0.3 * np.sin(2 * np.pi * x) + 0.5 * (x > 0.6) + noise
    v, p = 0.2 * np.cos(2 * np.pi * x), 1 + 0.8 * (x < 0.25)
    return np.stack([rho, rho * v, p / 0.4 + 0.5 * rho * v * v])


@pytest.mark.parametrize("flux", ["euler", "burgers"])
@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
@pytest.mark.parametrize("P", [1, 2, 3, 4, 5, 6])
def test_recorded_replayed_and_adjoint(acat, P, bc, flux):
    per = PER[P]
    for n in sorted({max(2 * P, 4), 2 * P + 3, per - 1, per, per + 1, 2 * per - 1, 255, 256, 257, 1000}):
        if n < 2 * P:
            continue
        nv = 3 if flux == "euler" else 1
        po, pg = both_problems(1, nv, n, flux, P, bc, 1.0 / n)
        u = np.ascontiguousarray(state(n, flux))
        dt = oracle.dt_cfl(po, u, 0.4)
        r = oracle.step1d(po, u, dt)
        ug, ws, dec = torch.from_numpy(u).cuda(), acat.workspace(pg), acat.Decisions(pg)
        ws.fill_(255)
        a = acat.step(pg, ug, dt, ws=ws, dec=dec)
        assert np.array_equal(a.cpu().numpy(), r["u"]), n
        for t, name in ((dec.order_x, "order"), (dec.psi1_x, "psi1"), (dec.alpha_x, "alpha")):
            assert np.array_equal(t.cpu().numpy(), r[name]), (n, name)
        want = np.bincount(r["order"], minlength=P + 1)[1:]
        counts = ws[:4 * P].view(torch.int32)
        assert counts.tolist() == want.tolist(), n
        ub = torch.from_numpy(np.random.default_rng(P).standard_normal(u.shape)).cuda()
        by_map = acat.step_adjoint_lists(pg, ug, dt, dec, ub, ws)
        by_orders = acat.step_adjoint(pg, ug, dt, dec, ub)
        assert torch.equal(by_map, by_orders), n
        ws.fill_(255)
        b = acat.step_replay(pg, ug, dt, dec, ws=ws)
        assert torch.equal(a, b) and counts.tolist() == want.tolist(), n
        assert torch.equal(acat.step_adjoint_lists(pg, ug, dt, dec, ub, ws), by_map), n
        assert torch.equal(acat.step(pg, ug, dt, ws=ws), a), n
        dtd = torch.zeros(1, dtype=torch.float64, device="cuda")
        c = acat.step_cfl(pg, ug, 0.4, dtd, ws=ws, dec=dec)
        assert counts.tolist() == want.tolist() and torch.equal(c, acat.step_replay(pg, ug, dtd, dec)), n
        if n <= 2 * per:
            dense = oracle.vjp_dense(po, u, ub.cpu().numpy(), dt, oracle.maps_of(po, r))
            err = np.abs(by_map.cpu().numpy() - dense).max()
            assert err <= 1e-11 * np.abs(dense).max(), (n, err)


def test_replayed_bad_order_is_taken_as_one_and_flagged(acat):
    n, P = 300, 3
    po, pg = both_problems(1, 3, n, "euler", P, "periodic", 1.0 / n)
    ug, dec = torch.from_numpy(np.ascontiguousarray(state(n, "euler"))).cuda(), acat.Decisions(pg)
    acat.step(pg, ug, 1e-4, dec=dec)
    dec.order_x[n - 1], dec.order_x[39] = 0, 4
    for t, v in ((dec.psi1_x, 0.5), (dec.alpha_x, 2.0)):
        t.fill_(v)
    acat.device_status()
    a = acat.step_replay(pg, ug, 1e-4, dec)
    assert acat.device_status() & 4
    dec.order_x[n - 1], dec.order_x[39] = 1, 1
    assert torch.equal(acat.step_replay(pg, ug, 1e-4, dec), a) and not acat.device_status() & 4
