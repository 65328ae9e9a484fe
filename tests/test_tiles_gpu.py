"""Tiles of the passes (lbm_params.tiles): 16-bit runs whose moment pass takes rectangular tiles and
whose collision takes packed rows, and x extents of each rectangular width, bitwise against rectangular
tiles everywhere; the request server against a run alone."""
import pytest

from paper_2606_29619_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
capi = pytest.importorskip("paper_2606_29619_amd.capi")


def _equal(a, b):
    assert torch.equal(a.populations(torch.float64), b.populations(torch.float64))
    for x, y in zip(a.moments(torch.float64), b.moments(torch.float64)):
        assert torch.equal(x, y)


# one cell past a 64-cell tile and one short of it, several tiles of every width
@pytest.mark.parametrize("nx", [5, 63, 65, 150, 192, 320, 384])
@pytest.mark.parametrize("storage", [capi.LBM_F16_SHIFTED, capi.LBM_BF16_SHIFTED])
@pytest.mark.parametrize("scheme", [capi.LBM_SCHEME_TWO_PASS, capi.LBM_SCHEME_LAGGED])
def test_tiles_of_16bit_runs_agree(nx, storage, scheme):
    w = workloads.random_porosity_3d(shape=(6, 9, nx), seed=nx, ell=3.0, nu=0.03, b=1e-4)
    kw = dict(storage=storage, scheme=scheme, shift=capi.LBM_SHIFT_POROUS)
    a = capi.Solver.from_workload(w, **kw)
    b = capi.Solver.from_workload(w, tiles=capi.LBM_TILES_RECTANGULAR, **kw)
    srv = capi.Server(pool_bytes=64 << 20, check_every=6)
    rid = srv.submit(w, storage=storage, scheme=scheme, tol=1e-300, max_steps=10 ** 6)
    other = workloads.random_porosity_3d(shape=(4, 5, 70), seed=1, ell=3.0, nu=0.03, b=1e-4)
    srv.submit(other, storage=storage, scheme=scheme, tol=1e-300, max_steps=10 ** 6)
    srv.progress(1)
    a.step(3)
    b.step(3)
    _equal(a, b)
    a.step(3)
    b.step(3)
    _equal(a, b)
    _equal(a, srv.solver(rid))
    srv.close()
