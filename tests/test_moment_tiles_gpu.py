"""Tiles of the 16-bit moment and lagged passes and of planes of few rows: bitwise the same cells whatever
tile updates them."""
import numpy as np
import pytest

from paper_2606_29619_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
capi = pytest.importorskip("paper_2606_29619_amd.capi")

STORAGE = {"f32": capi.LBM_F32, "f16": capi.LBM_F16_SHIFTED, "bf16": capi.LBM_BF16_SHIFTED}


def _equal(a, b):
    """Fields of a against those of b, repeated along y."""
    for x, y in ((a.populations(torch.float64), b.populations(torch.float64)),
                 *zip(a.moments(torch.float64), b.moments(torch.float64))):
        n = y.shape[-2]
        for k in range(0, x.shape[-2], n):
            assert torch.equal(x.narrow(-2, k, n), y)


# (nz, ny, nx): planes of one to three rows, which take wider moment tiles than the same plane repeated
# along y, and 16-bit rows that the moment pass packs or not
@pytest.mark.parametrize("shape", [(9, 1, 256), (9, 2, 256), (5, 3, 512), (4, 1, 192), (4, 2, 320),
                                   (6, 1, 100)])
@pytest.mark.parametrize("scheme", [capi.LBM_SCHEME_TWO_PASS, capi.LBM_SCHEME_LAGGED])
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_planes_of_few_rows(shape, scheme, storage):
    w = workloads.random_porosity_3d(shape=shape, seed=shape[2], ell=3.0, nu=0.03, b=1e-4)
    kw = dict(storage=STORAGE[storage], scheme=scheme, shift=1)
    small = capi.Solver.from_workload(w, **kw)
    for k in ("eps", "kappa", "forch"):
        setattr(w, k, np.tile(getattr(w, k), (1, 8, 1)))
    big = capi.Solver.from_workload(w, **kw)
    big.step(3)
    small.step(3)
    _equal(big, small)


# last and first extents of packed 16-bit moment tiles, and beyond
@pytest.mark.parametrize("nx", [3, 21, 22, 27, 28, 33, 53, 54, 66, 150])
@pytest.mark.parametrize("shift", [capi.LBM_SHIFT_WEIGHTS, capi.LBM_SHIFT_POROUS])
@pytest.mark.parametrize("scheme", [capi.LBM_SCHEME_TWO_PASS, capi.LBM_SCHEME_LAGGED])
def test_packed_moment_tiles_agree_with_rectangular(nx, shift, scheme):
    w = workloads.random_porosity_3d(shape=(6, 12, nx), seed=nx, ell=3.0, nu=0.03, b=1e-4)
    kw = dict(storage=capi.LBM_F16_SHIFTED, scheme=scheme, shift=shift)
    a = capi.Solver.from_workload(w, **kw)
    b = capi.Solver.from_workload(w, tiles=capi.LBM_TILES_RECTANGULAR, **kw)
    for steps in (3, 2):
        a.step(steps)
        b.step(steps)
        _equal(a, b)
