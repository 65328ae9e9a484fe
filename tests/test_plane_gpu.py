"""The one-launch D2Q9 step (lbm_params.passes) against the separate passes of the same library,
which evaluate the same expressions: bitwise equal populations and moments."""
import numpy as np
import pytest

from paper_2606_29619_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
capi = pytest.importorskip("paper_2606_29619_amd.capi")

STORAGE = {"f64": capi.LBM_F64, "f32": capi.LBM_F32, "f16": capi.LBM_F16_SHIFTED,
           "bf16": capi.LBM_BF16_SHIFTED}


def _workload(shape, solids, seed=5):
    ny, nx = shape
    w = workloads.random_porosity_2d(nx=nx, ny=ny, seed=seed, ell=3.0, nu=0.03, b=2e-4)
    w.RT, w.eta_eff, w.nu_eff_pow = 0.36, 0.02, -1
    if solids:  # scattered cells, single-cell corridors (one-sided stencils of every kind), a wall
        m = (np.random.default_rng(seed).random(w.shape) < 0.12).astype(np.uint8)
        m[:, 0, :] = 1
        m[0, -1, -1] = 0
        w.mask = m
    return w


def _equal(a, b):
    assert torch.equal(a.populations(torch.float64), b.populations(torch.float64))
    for x, y in zip(a.moments(torch.float64), b.moments(torch.float64)):
        assert torch.equal(x, y)


# (ny, nx): narrower than a tile and its rings along either axis (rings wrap several times), whole
# tiles, ragged tiles, the last size of the small tile and the first of the large one, a large plane
@pytest.mark.parametrize("shape", [(1, 256), (260, 1), (3, 90), (130, 2), (16, 16), (9, 31),
                                   (61, 67), (255, 257), (256, 256), (131, 1019)])
@pytest.mark.parametrize("storage,shift", [("f64", 0), ("f32", 0), ("f16", 1), ("bf16", 0)])
@pytest.mark.parametrize("solids", [False, True])
def test_one_launch_step_equals_separate_passes(shape, storage, shift, solids):
    if solids and min(shape) < 8:
        pytest.skip("no room for solid cells")
    w = _workload(shape, solids)
    kw = dict(storage=STORAGE[storage], shift=shift)
    a = capi.Solver.from_workload(w, **kw)
    b = capi.Solver.from_workload(w, passes=capi.LBM_PASSES_SEPARATE, **kw)
    assert a.nbytes > b.nbytes                      # the second population buffer
    ta, tb = a.step_timed(3), b.step_timed(3)       # ends in the swapped phase
    assert ta[0] == ta[1] == 0.0 and tb[0] > 0.0 and tb[1] > 0.0
    _equal(a, b)
    a.step(2)                                       # from the swapped phase, after a read
    b.step(2)
    assert a.residual().mass == b.residual().mass
    a.step(3)
    b.step(3)
    _equal(a, b)
    a.set_populations(b.populations(torch.float64), step=8)
    a.step(1)
    b.step(1)
    _equal(a, b)


def test_workspace_without_second_buffer_is_accepted():
    """The footprint of the separate passes is enough: such a run steps in separate passes."""
    w = _workload((61, 67), True)
    p, keep = capi.make_params(w.lattice, capi.LBM_F64, w.eps, w.kappa, w.forch, w.mask, RT=w.RT,
                               nu_f=w.nu_f, nu_eff_ref=w.nu_eff_ref, nu_eff_pow=w.nu_eff_pow,
                               eta_eff=w.eta_eff, b=w.b, rho0=w.rho0)
    p.passes = capi.LBM_PASSES_SEPARATE
    small = capi.lbm_footprint(p)
    p.passes = capi.LBM_PASSES_AUTO
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    h = capi.lbm_create(p, ws.data_ptr(), small, torch.cuda.current_stream().cuda_stream)
    ms = capi.lbm_step_timed(h, 3)
    capi.lbm_destroy(h)
    assert ms[0] > 0.0 and ms[1] > 0.0
    with pytest.raises(capi.LbmError) as ei:
        capi.lbm_create(p, ws.data_ptr(), small - 1, 0)
    assert ei.value.code == capi.LBM_ERR_WORKSPACE
