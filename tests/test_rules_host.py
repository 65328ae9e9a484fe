"""Rules by which the library chooses the kernels of a run, on the host (no GPU)."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2606_29619_amd import build, capi

STORAGES = [capi.LBM_F64, capi.LBM_F32, capi.LBM_F16_SHIFTED, capi.LBM_BF16_SHIFTED]
POP_BYTES = {capi.LBM_F64: 8, capi.LBM_F32: 4, capi.LBM_F16_SHIFTED: 2, capi.LBM_BF16_SHIFTED: 2}


def _second_buffer(shape, storage, solids=False, **kw):
    """Bytes that lbm_footprint counts beyond those of the separate passes."""
    nz, ny, nx = shape
    one = np.ones(shape)
    mask = np.zeros(shape, np.uint8) if solids else None
    sizes = []
    for passes in (capi.LBM_PASSES_AUTO, capi.LBM_PASSES_SEPARATE):
        p, keep = capi.make_params(capi.LBM_D2Q9 if nz == 1 else capi.LBM_D3Q27, storage, one, one, one,
                                   mask, passes=passes, **kw)
        sizes.append(capi.lbm_footprint(p))
    return sizes[0] - sizes[1]


@pytest.mark.parametrize("solids", [False, True])
@pytest.mark.parametrize("storage", STORAGES)
def test_thin_planes_step_in_separate_passes(storage, solids):
    """(ny, nx) of planes whose tiles would be mostly idle: separate passes, one buffer."""
    thin = [(1, 65536), (1, 262144)]
    if storage in (capi.LBM_F64, capi.LBM_F32):  # 16-bit: the separate passes idle as much along x
        thin += [(65536, 1), (262140, 1), (262140, 4)]
    for ny, nx in thin:
        assert _second_buffer((1, ny, nx), storage, solids) == 0, (ny, nx)


@pytest.mark.parametrize("solids", [False, True])
@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("shape", [(64, 128), (160, 320), (256, 256), (977, 1019), (1024, 1024),
                                   (1024, 1), (1024, 4)])
def test_planes_step_in_one_launch(shape, storage, solids):
    """A second population buffer, exactly."""
    n = 9 * shape[0] * shape[1] * POP_BYTES[storage]
    assert _second_buffer((1,) + shape, storage, solids) == (n + 255) // 256 * 256


def test_runs_without_a_second_buffer():
    shape = (1, 64, 128)
    z2, z3 = np.zeros((2,) + shape), np.zeros((3,) + shape)
    assert _second_buffer(shape, capi.LBM_F64, grad_eps=z2, hess_eps=z3) == 0
    assert _second_buffer(shape, capi.LBM_F64, picard_iters=2) == 0
    assert _second_buffer(shape, capi.LBM_F64, scheme=capi.LBM_SCHEME_LAGGED) == 0
    assert _second_buffer((1, 15, 17), capi.LBM_F64) == 0
    assert _second_buffer((8, 64, 64), capi.LBM_F64) == 0
    mask = np.zeros(shape, np.uint8)
    mask[:, 0] = mask[:, -1] = 1
    bt, bn = np.zeros(shape, np.uint8), np.zeros(shape, np.uint8)
    bt[:, 1], bn[:, 1] = capi.LBM_NODE_VELOCITY, capi.LBM_NORMAL_YM
    sizes = []
    for passes in (capi.LBM_PASSES_AUTO, capi.LBM_PASSES_SEPARATE):
        p, keep = capi.make_params(capi.LBM_D2Q9, capi.LBM_F64, np.ones(shape), np.ones(shape),
                                   np.ones(shape), mask, bc_type=bt, bc_normal=bn, passes=passes)
        sizes.append(capi.lbm_footprint(p))
    assert sizes[0] == sizes[1]


WRAPPER = r"""
#include "lbm_host.hpp"
// width (0: packed rows) and workgroups of the 16-bit moment tiles; width of the other tiles
extern "C" void moment_tiles(int nx, int ny, int nz, int pack, int lagged, int weights, int64_t out[2]) {
    const lbm::Tiling t = lbmh::moment_tiles(nx, ny, nz, true, pack, lagged, weights);
    out[0] = t.packed ? 0 : t.tx;
    out[1] = 8 * (int64_t)t.per;
}
extern "C" int rect_tile_x(int nx, int ny) { return lbmh::rect_tile_x(nx, ny); }
"""


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    """The tile rules of lbm_host.hpp, compiled for the host alone."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.hip").write_text(WRAPPER)
    subprocess.run([hipcc, "--offload-host-only", "-std=c++17", "-O1", "-fPIC", "-shared",
                    "-I", os.path.join(build.PKG, "csrc"), "-I", os.path.join(build.ROOT, "include"),
                    "-o", str(d / "rules.so"), str(d / "rules.hip")], check=True)
    lib = ctypes.CDLL(str(d / "rules.so"))

    def moment(nx, ny, nz, lagged=False, weights=False, pack=None):
        out = (ctypes.c_int64 * 2)()
        lib.moment_tiles(nx, ny, nz, int(nx % 64 != 0 if pack is None else pack), int(lagged),
                         int(weights), out)
        return out[0], out[1]

    return moment, lib.rect_tile_x


@pytest.mark.parametrize("lagged", [False, True])
def test_moment_tiles_of_narrow_rows(tiles, lagged):
    """16-bit D3Q27 rows much narrower than a tile are packed; the launch stays within the 2^32 threads
    that it may have at the largest grids of such rows."""
    moment, _ = tiles
    for nx in (1, 2, 3, 5, 9, 17):
        assert moment(nx, 192, 160, lagged)[0] == 0, nx
    for nx, ny, nz in ((1, 16384, 16383), (2, 8192, 16383), (3, 262140, 341)):
        assert nx * ny * nz < 2 ** 28 and 256 * moment(nx, ny, nz, lagged)[1] < 2 ** 32
    for nx in (37, 50, 70, 107, 150, 200, 220):
        assert moment(nx, 192, 160, lagged)[0] == 64, nx


@pytest.mark.parametrize("lagged", [False, True])
def test_moment_tiles_under_the_weight_shift(tiles, lagged):
    """No porosity in the decode: packed like FP32's where a fifth of the lanes would idle."""
    moment, _ = tiles
    for nx in (17, 33, 50, 66, 70, 100, 150):
        assert moment(nx, 192, 160, lagged, weights=True)[0] == 0, nx
    for nx in (60, 107, 120, 220, 250):
        assert moment(nx, 192, 160, lagged, weights=True)[0] == 64, nx


def test_tiles_of_planes_of_few_rows(tiles):
    """A plane of one to three rows leaves tiles of four rows mostly idle."""
    moment, rect = tiles
    for nx in (256, 512):
        for lagged in (False, True):
            assert moment(nx, 1, 4096, lagged)[0] == 256
    assert moment(512, 3, 2048, True)[0] == 256 and moment(512, 4, 2048, True)[0] == 64
    assert rect(192, 1) == 256 and rect(192, 4) == 64 and rect(448, 3) == 64
    for nx, tx in ((64, 64), (96, 128), (128, 128), (192, 64), (256, 256), (320, 64), (384, 128),
                   (448, 64), (512, 256)):
        for ny in (4, 64, 192):
            assert rect(nx, ny) == tx, (nx, ny)
