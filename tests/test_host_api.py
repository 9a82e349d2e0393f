"""The host side of the C ABI on the CPU: mhd_api.hip compiled for the host,
with the HIP runtime and the kernel launches replaced by stand-ins
(host_api.cpp).  Needs hipcc."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def api(tmp_path_factory):
    from paper_2604_12672_amd import build
    if shutil.which(build.HIPCC) is None and not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("host_api")
    obj, exe = str(d / "host_api.o"), str(d / "host_api")
    subprocess.run([build.HIPCC, "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-O1",
                    "-fPIC", "-std=c++17", "-c", os.path.join(HERE, "host_api.cpp"), "-o", obj], check=True)
    subprocess.run(["g++", obj, "-o", exe], check=True)

    def run(*args, zseg=None):
        env = dict(os.environ)
        env.pop("MHD_ZSEG", None)
        if zseg is not None:
            env["MHD_ZSEG"] = str(zseg)
        return subprocess.run([exe] + [str(a) for a in args], check=True, capture_output=True,
                              text=True, timeout=60, env=env).stdout.split()
    return run


def split(api, nx, ny, nz, precision, **kw):
    return dict(zip(("full", "share", "zseg", "blocks"),
                    map(int, api("split", nx, ny, nz, precision, **kw))))


# one to seven tiles with a long z: a march that leaves most of the CUs (256
# here, one FP64 or two split blocks each) without work takes that much longer
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nx,ny,nz", [(1, 1, 4096), (1, 1, 8192), (14, 14, 8192), (28, 14, 4096),
                                      (42, 14, 20000), (98, 14, 6000), (14, 14, 1000003)])
def test_tall_narrow_grid_fills_the_chip(api, nx, ny, nz, precision):
    s = split(api, nx, ny, nz, precision)
    slots = 256 * (1 + precision)
    tiles = -(-nx // 14) * -(-ny // 14)
    assert s["full"] == 0
    assert s["share"] == s["zseg"] <= -(-nz // (slots // tiles))
    assert s["blocks"] == tiles * -(-nz // s["share"])


# a launch holds fewer than 2^32 threads; a line of these cells has more tiles
# than that allows blocks of 512 threads
@pytest.mark.parametrize("nx,ny,nz,zseg", [(120000000, 1, 1, None), (536870911, 1, 2, None),
                                           (1, 117441000, 3, None), (30000000, 1, 4, 1)])
def test_launch_of_very_many_tiles(api, nx, ny, nz, zseg):
    assert split(api, nx, ny, nz, 1, zseg=zseg)["blocks"] * 512 < 2 ** 32


# the species and flag kernels: the same rule on their tiles and their slots
@pytest.mark.parametrize("tiles,nz,slots", [(1, 20000, 512), (1, 30000, 1024), (3, 90000, 1024),
                                            (7, 1000003, 2048)])
def test_segments_of_few_tiles_fill_the_chip(api, tiles, nz, slots):
    assert int(api("segment", tiles, nz, slots, 3)[0]) <= -(-nz // (slots // tiles))


# few lanes of a tile with a cell: the 16 planes the kernel had for every grid,
# where they leave enough blocks
@pytest.mark.parametrize("nx,ny,nz,planes", [
    (1, 1, 131072, 16), (1, 1, 131056, 8), (7, 5, 100000, 16), (16, 4, 131072, 16),
    (17, 4, 131072, 8), (1, 1, 32768, 8), (1, 1, 32760, 4), (192, 192, 192, 4), (256, 256, 256, 8),
    (64, 4, 1000000, 8)])
def test_planes_of_a_diffusion_block(api, nx, ny, nz, planes):
    assert int(api("dsegment", nx, ny, nz)[0]) == planes


# the background and the sources share one table: a call that fails leaves no
# half of its own values for the next one to upload, and no buffer behind
@pytest.mark.parametrize("what,times", [("malloc", 1), ("copy", 3), ("sync", 3)])
def test_failed_call_leaves_sources_and_background(api, what, times):
    failed, wrong, live = map(int, api("sources", what))
    assert (failed, wrong, live) == (times, 0, 0)


# creating a grid, the background, the sources (split precision and FP64) and
# the network: no exception leaves the C functions
def test_failed_host_allocation_is_an_error_code(api):
    calls, reached, thrown, missed, live = map(int, api("host_memory"))
    assert reached >= 2 * calls
    assert (thrown, missed, live) == (0, 0, 0)


# the ten buffers of the diffusion are there together or not at all, and the
# call after a failed one does not report its error again
def test_failed_allocation_of_a_diffusion_buffer(api):
    failed, missing, refused, live = map(int, api("diffusion"))
    assert (failed, missing, refused, live) == (10, 0, 0, 0)
