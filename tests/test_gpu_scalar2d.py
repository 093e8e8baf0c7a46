"""The 2D step of a scalar law at P = 1 and 2, whose flux blocks take fixed shares of
the class lists, and at P = 2 above 250000 corners tickets of two rounds and more: one
step against the oracle on both sides of the line and on grids of fewer rounds than
blocks, bit for bit, and the square-stencil variant."""
import numpy as np
import pytest

from gpu_helpers import both_problems
from test_gpu_parity import lockstep

pytestmark = pytest.mark.gpu


def data(nx, ny):
    rng = np.random.default_rng(nx + ny)
    X, Y = np.meshgrid((np.arange(nx) + 0.5) / nx, (np.arange(ny) + 0.5) / ny, indexing="xy")
    noise = 1e-3 * rng.standard_normal((ny, nx)) * (((X > 0.1) & (X < 0.2)) | ((Y > 0.7) & (Y < 0.8)))
    return (np.sin(2 * np.pi * X) * np.cos(2 * np.pi * Y) + 0.5 * (X > 0.6) + noise)[None].copy()


@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
@pytest.mark.parametrize("P,nx,ny", [(1, 16, 17), (1, 130, 95), (1, 700, 613), (2, 16, 17), (2, 130, 95),
                                     (2, 499, 499), (2, 501, 500), (2, 733, 610)])
def test_scalar_step_equals_the_oracle(acat, P, nx, ny, bc):
    for flags in (0, acat.FLAG_SQUARE_2D) if nx < 600 else (0,):
        po, pg = both_problems(2, 1, nx, "advection", P, bc, 1.0 / nx, ny=ny, dy=1.0 / ny, ax=0.8, ay=-0.6,
                               flags=flags)
        lockstep(acat, po, pg, data(nx, ny), 0.4, 1, label=f"advection2d P={P} {bc} {nx}x{ny} flags={flags}")
