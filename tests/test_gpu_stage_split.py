"""The stage kernel's split of the work over the blocks: whole columns and
segments of planes, segments of one plane, grids smaller than a tile and the
shortest z axes.  The state does not depend on the split (bit for bit against
segments of one and of three planes) and agrees with the oracle: FP64 to
1e-10 per field, the bound of the other parity tests, split precision to its
1e-5."""
import os

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


def run(mhd, w, dts, precision, zseg=None):
    if zseg is not None:
        os.environ["MHD_ZSEG"] = str(zseg)
    try:
        g = mhd.Grid(w.params, precision=precision)
    finally:
        os.environ.pop("MHD_ZSEG", None)
    g.load(w)
    for dt in dts:
        g.step(dt)
    out, info = g.get_state(), g.launch_info()
    g.close()
    return out, info


# 306 tiles: more than the CUs of the chip, so FP64 takes whole columns first
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nx,ny,nz,bcz,eos", [
    (239, 225, 5, 0, 0), (240, 236, 3, 1, 0), (226, 239, 4, 1, 1),
    (15, 14, 1, 0, 0), (14, 29, 2, 1, 0), (13, 1, 3, 0, 1), (1, 28, 2, 1, 0), (3, 2, 1, 0, 0)])
def test_split_of_the_work(mhd, nx, ny, nz, bcz, eos, precision):
    print(f"case {nx}x{ny}x{nz} bcz={bcz} eos={eos} prec={precision}", flush=True)
    w = wl.smooth_box(nx, ny, nz, bcz=bcz, eos=eos)
    o = orc.Oracle(w.params, **w.extras())
    ref = w.state()
    dts = [0.5 * o.compute_dt(ref, 0.3)] * 2
    for dt in dts:
        o.step(ref, dt)
    out, info = run(mhd, w, dts, precision)
    if nx > 200 and precision == 0:
        assert info["zseg"] == nz and info["blocks"] < 306
    tol = 1e-10 if precision == 0 else 1e-5
    for k in ("U", "Bx", "By", "Bz"):
        a, b = np.asarray(out[k]), ref[k]
        assert np.sqrt(np.sum((a - b) ** 2)) <= tol * np.sqrt(np.sum(b * b)) + 1e-300, k
    for zseg in (1, 3):
        cut, cinfo = run(mhd, w, dts, precision, zseg)
        assert cinfo["zseg"] == min(zseg, nz)
        for k in ("U", "Bx", "By", "Bz"):
            assert np.array_equal(out[k], cut[k]), (k, zseg)
