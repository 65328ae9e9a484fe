"""lbm_moments where the velocity correction writes the caller's arrays: every output form against the
FP64 superficial one, and that one against the CPU oracle and the statistics."""
import ctypes

import numpy as np
import pytest

from paper_2606_29619_amd import workloads
from tests.oracle_cases import from_workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
capi = pytest.importorskip("paper_2606_29619_amd.capi")

FP64_TOL = 1e-12


def _box(D, solids):
    if D == 2:
        w = workloads.random_porosity_2d(nx=70, ny=21, seed=4, ell=3.0, nu=0.03, b=1e-4)
    else:
        w = workloads.random_porosity_3d(shape=(7, 9, 40), seed=4, ell=3.0, nu=0.03, b=1e-4)
    if solids:
        w.mask = (np.random.default_rng(1).random(w.shape) < 0.1).astype(np.uint8)
    return w


@pytest.mark.parametrize("D", [2, 3])
@pytest.mark.parametrize("solids", [False, True])
@pytest.mark.parametrize("scheme", [capi.LBM_SCHEME_TWO_PASS, capi.LBM_SCHEME_LAGGED])
@pytest.mark.parametrize("storage", [capi.LBM_F64, capi.LBM_F32, capi.LBM_F16_SHIFTED])
def test_output_forms(D, solids, scheme, storage):
    w = _box(D, solids)
    s = capi.Solver.from_workload(w, storage=storage, scheme=scheme)
    s.step(3)
    rho, v = s.moments(torch.float64)
    eps = torch.tensor(np.asarray(w.eps).reshape(s.shape), device="cuda")
    if storage != capi.LBM_F64:
        eps = eps.float()  # the quotient is formed in the arithmetic type
    u = (v.to(eps.dtype) / eps).double()
    ri, vi = s.moments(torch.float64, intrinsic=True)
    assert torch.equal(ri, rho) and torch.equal(vi, u)
    for intrinsic, want in ((False, v), (True, u)):
        r32, v32 = s.moments(torch.float32, intrinsic=intrinsic)
        assert torch.equal(r32, rho.float()) and torch.equal(v32, want.float())
    # either output may be left out; the other is written, nothing beyond it
    for which in (0, 1):
        out = torch.full((rho.numel() if which == 0 else v.numel(),), 7.0, dtype=torch.float64,
                         device="cuda")
        guard = torch.cat([out, torch.full((64,), 7.0, dtype=torch.float64, device="cuda")])
        ptrs = [0, 0]
        ptrs[which] = guard.data_ptr()
        capi.lbm_moments(s.handle, *ptrs, capi.LBM_DTYPE_F64, capi.LBM_VELOCITY_SUPERFICIAL)
        assert torch.equal(guard[:out.numel()], (rho if which == 0 else v).reshape(-1))
        assert torch.equal(guard[out.numel():], torch.full((64,), 7.0, dtype=torch.float64, device="cuda"))
    # reading changes nothing: the same reads again, and the steps that follow
    assert all(torch.equal(a, b) for a, b in zip(s.moments(torch.float64), (rho, v)))
    t = capi.Solver.from_workload(w, storage=storage, scheme=scheme)
    t.step(3)
    s.step(2)
    t.step(2)
    assert torch.equal(s.populations(torch.float64), t.populations(torch.float64))
    st = s.residual()
    speed = s.moments(torch.float64)[1].pow(2).sum(0).sqrt().max().item()
    assert abs(st.vmax - speed) <= 1e-15 * speed


@pytest.mark.parametrize("D", [2, 3])
@pytest.mark.parametrize("case", ["box", "solids", "analytic"])
@pytest.mark.parametrize("lagged", [0, 1])
def test_matches_oracle(D, case, lagged):
    """After steps, and (lagged) with the history gone after populations are set."""
    if case == "analytic":
        w = workloads.sine_porosity(D, shape=(1, 18, 24) if D == 2 else (8, 10, 24))
        extra = dict(grad_eps=w.grad_eps, hess_eps=w.hess_eps)
    else:
        w, extra = _box(D, case == "solids"), {}
    s = capi.Solver.from_workload(w, storage=capi.LBM_F64, scheme=lagged)
    o = from_workload(w, lagged=lagged, **extra)
    for steps in (3, 2):
        s.step(steps)
        o.step(steps)
        ro, vo, _ = o.moments()
        for got, ref in zip(s.moments(torch.float64), (ro, vo)):
            assert np.abs(got.cpu().numpy() - ref).max() <= FP64_TOL * np.abs(ref).max()
    f = s.populations(torch.float64)
    two = capi.Solver.from_workload(w, storage=capi.LBM_F64)
    for x in (s, two):
        x.set_populations(f, step=5)
    for a, b in zip(s.moments(torch.float64), two.moments(torch.float64)):
        assert torch.equal(a, b)  # without a previous step the lagged scheme reads as the two-pass one
