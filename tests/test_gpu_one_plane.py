"""The stage of a grid of one plane has kernels of its own.  A state that
does not vary along z has, on a grid of one plane, bit for bit the planes it
has on a grid of four, whose steps the general kernels take: every EOS,
precision and optional feature, on one cell along x, a tile's interior (14
cells a side) and one more, ragged tiles, and more tiles than the chip has
CUs.  The stage takes the difference of the fluxes through a cell's z-faces
first, which is zero on both grids, so nothing is left to a tolerance.  The
species kernel leaves the z-faces out on one plane and adds the upper face's
term to a sum that began with the lower's on four: three roundings a stage of
sums that the time step bounds by the value itself, nine stages, so 128 units
of the largest value's last place."""
import numpy as np
import pytest

from oracle import orc
from paper_2604_12672_amd import workloads as wl

pytestmark = pytest.mark.gpu

# wavevectors without a z component: the forcing does not vary along z either
FMODES = np.array([[1, 0, 0, 0.0, 0.3, 0.1, 0.4], [0, -2, 0, 0.2, 0.0, -0.2, 1.1]])


@pytest.fixture(scope="module")
def mhd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_12672_amd import mhd as m
    m.load()
    return m


def stacked(w, n):
    """The workload w of one plane on a grid of n planes."""
    rep = lambda a: None if a is None else np.ascontiguousarray(np.repeat(a, n, axis=a.ndim - 3))
    row = lambda a: None if a is None else np.ascontiguousarray(np.repeat(a, n, axis=-1))
    return wl.Workload(w.name, dict(w.params, nz=n), rep(w.U), rep(w.Bx), rep(w.By), rep(w.Bz),
                       T=rep(w.T), bg_cc=row(w.bg_cc), bg_fz=row(w.bg_fz), heat=row(w.heat),
                       fmodes=w.fmodes)


def run(mhd, w, dts, precision):
    g = mhd.Grid(w.params, precision=precision)
    g.load(w)
    for dt in dts:
        g.step(dt)
    out = g.get_state(with_T=bool(w.params["eos"]))
    if w.params.get("nspecies"):
        out["X"] = g.get_species()
    d = g.diagnostics()
    g.close()
    return out, d


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("eos", [0, 1])
@pytest.mark.parametrize("extra", [False, True])
@pytest.mark.parametrize("nx,ny", [(1, 5), (14, 15), (29, 41), (242, 239)])
def test_one_plane_against_four(mhd, nx, ny, extra, eos, precision):
    print(f"case {nx}x{ny} extra={extra} eos={eos} prec={precision}", flush=True)
    w = wl.smooth_box(nx, ny, 1, eos=eos, blast=(4.0, 0.3) if extra else None)
    w.params = dict(w.params, recon=orc.RECON_PPH, rk_order=3) if extra else w.params
    if extra:
        w.params = dict(w.params, flatten=1)
        w.fmodes, w.heat = FMODES, np.array([0.02])
        w = wl.add_species(w, 2)
    o = orc.Oracle(w.params, **w.extras())
    dts = [0.5 * o.compute_dt(w.state(), 0.3)] * 3
    one, d1 = run(mhd, w, dts, precision)
    four, d4 = run(mhd, stacked(w, 4), dts, precision)
    for z in range(4 if extra else 0):
        assert np.abs(one["X"][:, 0] - four["X"][:, z]).max() <= 128 * 2.0 ** -52 * one["X"].max()
    for k in (k for k in one if k != "X"):
        for z in range(4):
            assert np.array_equal(one[k][..., 0, :, :], four[k][..., z, :, :]), (k, z)
    assert 4 * d1["newton_iters"] == d4["newton_iters"]
    assert d1["newton_max"] == d4["newton_max"] and d1["error_flags"] == d4["error_flags"] == 0
