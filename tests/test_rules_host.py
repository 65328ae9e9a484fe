"""Rules by which the library chooses the kernels of a run, on the host (no GPU)."""
import numpy as np
import pytest

from paper_2606_29619_amd import capi

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
