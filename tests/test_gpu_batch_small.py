"""A batch of very many very small problems, without a launch table: it goes by
passes, one launch per order class, and equals the steps of the single problems bit
for bit, as a smaller batch of the same problems by tiles does."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def state(flux, n, seed):
    rng = np.random.default_rng(seed)
    x = (np.arange(n) + 0.5) / n
    if flux == "burgers":
        return (0.5 + np.sin(2 * np.pi * x) + 0.1 * rng.standard_normal(n) * (x > 0.6))[None]
    rho = 1.0 + 0.2 * np.sin(2 * np.pi * x) + 0.5 * (x > 0.5)
    return workloads.euler1d_conserved(rho, 0.1 * rng.standard_normal(n) * (x > 0.4), 1.0 + 0.5 * (x < 0.3))


@pytest.mark.parametrize("flux", ["euler", "burgers"])
def test_small_problems(acat, flux):
    kinds = [(n, P, bc) for n in (8, 9, 17, 31, 40) for P in (1, 2, 3, 4) for bc in ("periodic", "transmissive")]
    us = [np.ascontiguousarray(state(flux, n, k)) for k, (n, _, _) in enumerate(kinds)]
    res = {}
    for copies in (200, 2):
        ks = kinds * copies
        batch = acat.Batch([k[0] for k in ks], [k[1] for k in ks], [k[2] for k in ks], [1.0 / k[0] for k in ks],
                           flux=flux, nvar=us[0].shape[0])
        u = torch.from_numpy(np.concatenate(us * copies, axis=1)).cuda()
        dt = torch.empty(len(ks), dtype=torch.float64, device="cuda")
        batch.cfl_dt(u, 0.4, dt)
        used = dt.clone()
        acat.profile(True)
        out = batch.step_cfl(u, dt, 0.4)
        again = batch.step(u, used)
        ran = acat.profile_read()
        acat.profile(False)
        assert ("classify_b" in ran, "step_b" in ran) == ((True, False) if copies == 200 else (False, True)), ran
        assert torch.equal(out, again)
        res[copies] = (used, out, dt)
    many, few = res[200], res[2]
    cells, probs = few[1].shape[1], len(few[0])
    for k in range(100):
        assert torch.equal(many[1][:, k * cells:(k + 1) * cells], few[1]), k
        assert torch.equal(many[0][k * probs:(k + 1) * probs], few[0])
        assert torch.equal(many[2][k * probs:(k + 1) * probs], few[2])
    c0 = 0
    for k, (n, P, bc) in enumerate(kinds):
        prob = acat.Problem(dim=1, nvar=us[0].shape[0], nx=n, flux=flux, P=P, bc=bc, dx=1.0 / n)
        single = acat.step(prob, torch.from_numpy(us[k]).cuda(), few[0][k:k + 1])
        assert torch.equal(few[1][:, c0:c0 + n], single), (n, P, bc)
        c0 += n
