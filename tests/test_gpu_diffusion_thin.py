"""Thermal diffusion on grids that fill a few lanes of a tile, whose blocks
take 16 planes: both forms against the oracle, walls and a ragged end, to
the bound of the other diffusion tests (rel L2 <= 1e-9 for E and T, the level
at which the Newton solves of the two sides stop)."""
import numpy as np
import pytest

from oracle import orc
from paper_2604_12672_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mhd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_12672_amd import mhd as m
    m.load()
    return m


def rel_l2(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("nx,ny,nz,bcz", [(1, 1, 131072, 0), (3, 2, 131085, 1)])
def test_thin_grid(mhd, nx, ny, nz, bcz, mode):
    print(f"case diffusion {nx}x{ny}x{nz} bcz={bcz} mode={mode}", flush=True)
    rng = np.random.default_rng(15)
    p = wl.gasrad_params(nx, ny, nz, bcz=bcz)
    shape = (nz, ny, nx)
    rho = 10.0 ** rng.uniform(-1, 1, size=shape)
    T = 10.0 ** rng.uniform(6, 7, size=shape)
    U = np.zeros((5,) + shape)
    U[0], U[4] = rho, rho * wl.gasrad_forward(p, rho, T)[1]
    B = np.zeros(shape)
    Bz = np.zeros((nz + 1 if bcz else nz, ny, nx))
    ref = {"U": U.copy(), "Bx": B.copy(), "By": B.copy(), "Bz": Bz.copy(), "T": T.copy()}
    kramers = dict(kappa0=0.2, alpha=1.0, beta=-3.5)
    op, o = orc.opacity(**kramers), orc.Oracle(p)
    dt = 25.0 * o.parabolic_dt(rho, T, op)
    o.diffuse(ref, dt, 7, op, mode=mode)
    g = mhd.Grid(p)
    g.set_state(U, B, B, Bz, T)
    g.set_opacity(**kramers)
    assert g.diffuse(dt, 7, mode) == 7
    out = g.get_state(with_T=True)
    g.close()
    assert rel_l2(out["U"][4], ref["U"][4]) < 1e-9
    assert rel_l2(out["T"], ref["T"]) < 1e-9
    np.testing.assert_array_equal(out["U"][:4], U[:4])
