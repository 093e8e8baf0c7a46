"""The 1D adjoint with the workspace of a step that recorded nothing, which leaves no
class map in it: wrong results, as documented, but nothing outside the buffers is read.
A map of values that are no class gives no interface a contribution: with the
contributions' buffer cleared the adjoint is ubar itself."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
@pytest.mark.parametrize("value", [6, 127, 128, 255])
def test_a_map_of_no_classes_contributes_nothing(acat, value, bc):
    for n in (12, 40, 700):
        prob = acat.Problem(dim=1, nvar=1, nx=n, flux="burgers", P=6, bc=bc, dx=1.0 / n)
        u = torch.sin(torch.arange(n, dtype=torch.float64, device="cuda") / n)[None].contiguous()
        dec, ws, aws = acat.Decisions(prob), acat.workspace(prob), acat.adjoint_workspace(prob)
        acat.step(prob, u, 1e-3, dec=dec)
        ws.fill_(value)
        acat.step(prob, u, 1e-3, ws=ws)
        aws.zero_()
        ub = torch.cos(3.0 * u)
        assert torch.equal(acat.step_adjoint_lists(prob, u, 1e-3, dec, ub, ws, ws=aws), ub), n
