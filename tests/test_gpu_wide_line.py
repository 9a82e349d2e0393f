"""A line of more tiles than a launch holds blocks of the split-precision stage
kernel (2^32 threads): some blocks take two.  The state repeats along the
line and the cell size is the short line's, so each of its copies is bit for
bit the short line after the same steps."""
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


def test_line_of_many_tiles(mhd):
    import torch
    n, copies = 1000001, 128
    w = wl.smooth_box(n, 1, 1)
    dt = 0.1 / n
    state = {k: torch.tensor(np.ascontiguousarray(getattr(w, k)), device="cuda")
             for k in ("U", "Bx", "By", "Bz")}

    def run(params, st):
        g = mhd.Grid(params, precision=mhd.PREC_SPLIT)
        info = g.launch_info()
        g.set_state(st["U"], st["Bx"], st["By"], st["Bz"])
        for _ in range(2):
            g.step(dt)
        out = g.get_state({k: torch.empty_like(v) for k, v in st.items()})
        g.close()
        return out, info

    short, info = run(w.params, state)
    tiles = -(-n // 14)
    assert info["blocks"] == tiles
    print("line of", copies * n, "cells", flush=True)
    hi = (float(copies) * w.params["hi"][0],) + tuple(w.params["hi"][1:])
    long, info = run(dict(w.params, nx=copies * n, hi=hi),
                     {k: v.repeat(*([1] * (v.dim() - 1) + [copies])) for k, v in state.items()})
    assert info["blocks"] * 512 < 2 ** 32 < -(-copies * n // 14) * 512
    for k in state:
        assert not torch.equal(short[k], state[k]) or k == "Bx"
        a = long[k].view(*long[k].shape[:-1], copies, n)
        assert bool((a == short[k].unsqueeze(-2)).all()), k
