"""A super step that takes its stage count from the parabolic limit starts from
the values the limit's kernel stores; one with a given count from those of a
kernel of its own.  With the same count the two are the same bit for bit:
both forms, with and without a stored temperature guess, grids of a few
cells, one block's cells and one more, and more cells than the blocks of the
reduction hold in one pass (2048 of 256)."""
import numpy as np
import pytest

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


def run(mhd, w, T, factor, nsts, mode):
    g = mhd.Grid(w.params)
    g.set_state(w.U, w.Bx, w.By, w.Bz, T)
    g.set_opacity(kappa0=0.2, alpha=1.0, beta=-3.5)
    used = g.diffuse(factor * g.parabolic_dt(), nsts, mode)
    out = g.get_state(with_T=True)
    g.close()
    return out, used


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("guess", [False, True])
@pytest.mark.parametrize("nx,ny,nz,bcz", [(3, 2, 1, 0), (16, 16, 1, 0), (257, 1, 1, 0),
                                          (13, 9, 7, 1), (97, 90, 67, 0)])
def test_start_from_the_limit(mhd, nx, ny, nz, bcz, guess, mode):
    print(f"case {nx}x{ny}x{nz} bcz={bcz} guess={guess} mode={mode}", flush=True)
    w = wl.smooth_box(nx, ny, nz, bcz=bcz, eos=1)
    T = w.T if guess else None
    auto, used = run(mhd, w, T, 10.3, 0, mode)
    given, again = run(mhd, w, T, 10.3, used, mode)
    assert used == again >= 3
    for k in auto:
        assert np.array_equal(auto[k], given[k]), k
