"""Solid cells at wave and tile edges of every rectangular tile width, and in planes narrower than the
tiles of the one-launch D2Q9 step."""
import numpy as np
import pytest

from paper_2606_29619_amd import workloads
from tests.oracle_cases import from_workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
capi = pytest.importorskip("paper_2606_29619_amd.capi")

FP64_TOL = 1e-12


# rows of 256 cells take 256 x 1 tiles, of 384 128 x 2, of 192 64 x 4, of 512 two tiles of 256 x 1
@pytest.mark.parametrize("lagged", [0, 1])
@pytest.mark.parametrize("nx", [192, 256, 384, 512])
def test_solids_at_wave_edges(nx, lagged):
    w = workloads.random_porosity_3d(shape=(6, 7, nx), seed=9, ell=3.0, nu=0.05, b=1e-4)
    m = np.zeros(w.shape, np.uint8)
    for k, x in enumerate([x for e in range(64, nx, 64) for x in (e - 1, e)] + [0, nx - 1]):
        m[(2 * k) % 6, (3 * k) % 7, x] = 1
    m[3, 2:5, 96:99] = 1
    w.mask = m
    s = capi.Solver.from_workload(w, storage=capi.LBM_F64, scheme=lagged)
    o = from_workload(w, lagged=lagged)
    for steps in (5, 3):  # the swapped and the natural phase next
        s.step(steps)
        o.step(steps)
        f, (rho, v) = s.populations(torch.float64), s.moments(torch.float64)
        ro, vo, _ = o.moments()
        for got, ref in ((f, o.populations()), (rho, ro), (v, vo)):
            got = got.cpu().numpy()
            assert np.abs(got - ref).max() <= FP64_TOL * np.abs(ref).max()


@pytest.mark.parametrize("shape", [(1, 256), (260, 1), (3, 90), (130, 2), (7, 300), (400, 5)])
@pytest.mark.parametrize("storage,shift", [(capi.LBM_F64, 0), (capi.LBM_F32, 0),
                                           (capi.LBM_F16_SHIFTED, 1), (capi.LBM_BF16_SHIFTED, 0)])
def test_narrow_planes_with_solids(shape, storage, shift):
    ny, nx = shape
    w = workloads.random_porosity_2d(nx=nx, ny=ny, seed=6, ell=3.0, nu=0.03, b=2e-4)
    w.eta_eff, w.nu_eff_pow = 0.02, -1
    w.mask = (np.random.default_rng(6).random(w.shape) < 0.08).astype(np.uint8)
    kw = dict(storage=storage, shift=shift)
    a = capi.Solver.from_workload(w, **kw)
    b = capi.Solver.from_workload(w, passes=capi.LBM_PASSES_SEPARATE, **kw)
    assert a.step_timed(1)[0] == 0.0 and b.step_timed(1)[0] > 0.0
    for steps in (2, 3):
        a.step(steps)
        b.step(steps)
        assert torch.equal(a.populations(torch.float64), b.populations(torch.float64))
        for x, y in zip(a.moments(torch.float64), b.moments(torch.float64)):
            assert torch.equal(x, y)
