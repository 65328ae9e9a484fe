"""Rounding of the 16-bit storage forms.  A population v is stored as (v - sigma) scaled by a power of two:
FP16 storage rounds the exact difference once, BF16 storage the FP32 difference."""
import numpy as np
import pytest

from paper_2606_29619_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
capi = pytest.importorskip("paper_2606_29619_amd.capi")
oracle = pytest.importorskip("oracle")


@pytest.mark.parametrize("D", [2, 3])
def test_fp16_storage_rounds_once(D):
    w = workloads.uniform_box(D=D, n=64 if D == 2 else 16)
    s = capi.Solver.from_workload(w, storage=capi.LBM_F16_SHIFTED, shift=capi.LBM_SHIFT_WEIGHTS)
    c, _ = oracle.lattice(D)
    f32 = np.float32
    wi = np.array([np.prod([f32(2 / 3) if x == 0 else f32(1 / 6) for x in row[:D]], dtype=f32)
                   for row in np.asarray(c)], f32)
    inv = np.array([4096.0 * np.prod([1.5 if x == 0 else 6.0 for x in row[:D]]) for row in np.asarray(c)])
    scale = 2.0 ** np.floor(np.log2(inv))
    rng = np.random.default_rng(2)
    shape = (s.Q,) + s.shape
    col = (slice(None),) + (None,) * 3
    # about rho0 w_I: half of them a random distance away, half close to the middle between two FP16
    # values, where rounding to FP32 first moves some across it
    d = rng.uniform(-0.9, 0.9, shape) * wi[col]
    mid = np.float16(d * scale[col]).astype(np.float64) + 0.5 * np.spacing(
        np.abs(np.float16(d * scale[col]))).astype(np.float64)
    d = np.where(rng.random(shape) < 0.5, d, mid / scale[col] * (1 + rng.uniform(-1e-7, 1e-7, shape)))
    v = (wi[col].astype(np.float64) + d).astype(f32)
    s.set_populations(torch.tensor(v, device="cuda"))
    exact = (v.astype(np.float64) - wi[col].astype(np.float64)) * scale[col]
    raw = exact.astype(np.float16)
    twice = exact.astype(f32).astype(np.float16)
    got = s.populations(torch.float64).cpu().numpy()
    want = raw.astype(np.float64) / scale[col] + wi[col].astype(np.float64)
    print("differ where rounded twice:", int((raw != twice).sum()), flush=True)
    assert np.array_equal(got, want)


# runs whose solo and batched kernels are compiled apart; enough cells and steps that a population
# rounded otherwise by one of them shows
@pytest.mark.parametrize("D", [2, 3])
@pytest.mark.parametrize("solids", [False, True])
@pytest.mark.parametrize("scheme", [capi.LBM_SCHEME_TWO_PASS, capi.LBM_SCHEME_LAGGED])
@pytest.mark.parametrize("shift", [capi.LBM_SHIFT_WEIGHTS, capi.LBM_SHIFT_POROUS])
def test_fp16_runs_do_not_depend_on_their_kernels(D, solids, scheme, shift):
    if D == 2:
        w = workloads.random_porosity_2d(nx=500, ny=420, seed=3, ell=6.0, nu=0.03, b=1e-4)
    else:
        w = workloads.random_porosity_3d(shape=(40, 48, 100), seed=3, ell=6.0, nu=0.03, b=1e-4)
    if solids:
        w.mask = (np.random.default_rng(3).random(w.shape) < 0.05).astype(np.uint8)
    kw = dict(storage=capi.LBM_F16_SHIFTED, scheme=scheme, shift=shift)
    runs = [capi.Solver.from_workload(w, **kw),
            capi.Solver.from_workload(w, tiles=capi.LBM_TILES_RECTANGULAR, **kw),
            capi.Solver.from_workload(w, passes=capi.LBM_PASSES_SEPARATE, **kw)]
    srv = capi.Server(pool_bytes=256 << 20, check_every=30)
    rid = srv.submit(w, tol=1e-300, max_steps=10 ** 6, **kw)
    srv.progress(1)
    f = srv.solver(rid).populations(torch.float64)
    for s in runs:
        s.step(30)
        assert torch.equal(s.populations(torch.float64), f)
    srv.close()
