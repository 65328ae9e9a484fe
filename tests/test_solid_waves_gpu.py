"""Solid cells at the edges of waves and tiles: every pass chooses its solid-aware code per wave of 64
cells, so cells next to a solid across a wave, tile or periodic edge must be found.  FP64 against the
CPU oracle, both schemes, rectangular and packed tiles."""
import numpy as np
import pytest

from paper_2606_29619_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
capi = pytest.importorskip("paper_2606_29619_amd.capi")
oracle = pytest.importorskip("oracle")

FP64_TOL = 1e-12


@pytest.mark.parametrize("lagged", [0, 1])
@pytest.mark.parametrize("nx", [320, 333])
def test_solids_at_wave_edges_match_oracle(nx, lagged):
    w = workloads.random_porosity_3d(shape=(6, 7, nx), seed=9, ell=3.0, nu=0.05, b=1e-4)
    m = np.zeros(w.shape, np.uint8)
    for k, x in enumerate((0, 63, 64, 127, 192, 255, 256, nx - 1)):
        m[(2 * k) % 6, (3 * k) % 7, x] = 1
    m[3, 2:5, 96:99] = 1
    w.mask = m
    s = capi.Solver.from_workload(w, storage=capi.LBM_F64, scheme=lagged)
    o = oracle.Oracle(oracle.OracleConfig(D=3, eps=w.eps, kappa=w.kappa, cf=w.forch, mask=m,
                                          nu_f=w.nu_f, nu_eff_ref=w.nu_eff_ref, b=w.b,
                                          lagged=lagged))
    for steps in (5, 3):  # the swapped and the natural phase next
        s.step(steps)
        o.step(steps)
        f, (rho, v) = s.populations(torch.float64), s.moments(torch.float64)
        ro, vo, _ = o.moments()
        for got, ref in ((f, o.populations()), (rho, ro), (v, vo)):
            got = got.cpu().numpy()
            assert np.abs(got - ref).max() <= FP64_TOL * np.abs(ref).max()
