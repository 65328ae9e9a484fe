"""Population accesses of large runs.  Runs whose working set fits the Infinity Cache access their
populations through the caches; larger ones stream them past the caches in some or all passes, so the
small grids of the other tests do not reach those kernels.  A periodic run repeated along z until its set is
too large evolves like the run itself, cell by cell and bit for bit, with other kernels."""
import numpy as np
import pytest

from paper_2606_29619_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
capi = pytest.importorskip("paper_2606_29619_amd.capi")

STORAGE = {"f64": capi.LBM_F64, "f32": capi.LBM_F32, "f16": capi.LBM_F16_SHIFTED,
           "bf16": capi.LBM_BF16_SHIFTED}
# bytes that a D3Q27 cell of a two-pass step works on, and the largest set that is kept in the cache
CELL_BYTES = {"f64": 27 * 8 + 11 * 8, "f32": 27 * 4 + 11 * 4, "f16": 27 * 2 + 11 * 4,
              "bf16": 27 * 2 + 11 * 4}
CACHED_SET = 240 << 20


def _base(nx, solids, seed=3):
    w = workloads.random_porosity_3d(shape=(16, 48, nx), seed=seed, ell=3.0, nu=0.03, b=1e-4)
    w.eta_eff = 0.02
    if solids:
        m = (np.random.default_rng(seed).random(w.shape) < 0.01).astype(np.uint8)
        m[3:9, 10:30, 5:40] = 1
        w.mask = m
    return w


def _repeated(w, axis, times):
    big = workloads.Workload(**w.__dict__)
    reps = [1, 1, 1]
    reps[axis] = times
    for k in ("eps", "kappa", "forch", "mask", "bc_type", "bc_normal", "bc_density"):
        a = getattr(w, k, None)
        if a is not None:
            setattr(big, k, np.tile(a, reps))
    for k in ("bc_velocity", "v_init"):
        a = getattr(w, k, None)
        if a is not None:
            setattr(big, k, np.tile(a, [1] + reps))
    return big


def _times(w, storage):
    return CACHED_SET // (CELL_BYTES[storage] * w.cells) + 2


def _assert_repeats(big, small, axis):
    for a, b in ((big.populations(torch.float64), small.populations(torch.float64)),
                 *zip(big.moments(torch.float64), small.moments(torch.float64))):
        d = axis - 3 + a.dim()
        n = b.shape[d]
        for k in range(0, a.shape[d], n):
            assert torch.equal(a.narrow(d, k, n), b)


@pytest.mark.parametrize("solids", [False, True])
@pytest.mark.parametrize("scheme", [capi.LBM_SCHEME_TWO_PASS, capi.LBM_SCHEME_LAGGED])
@pytest.mark.parametrize("nx", [64, 70])  # rows of whole cache lines and ragged rows
@pytest.mark.parametrize("storage,shift", [("f64", 0), ("f32", 0), ("f16", 0), ("bf16", 1)])
def test_large_runs_repeat_small_ones(storage, shift, nx, scheme, solids):
    w = _base(nx, solids)
    kw = dict(storage=STORAGE[storage], shift=shift, scheme=scheme, passes=capi.LBM_PASSES_SEPARATE)
    big = capi.Solver.from_workload(_repeated(w, 0, _times(w, storage)), **kw)
    small = capi.Solver.from_workload(w, **kw)
    for steps in (3, 2):  # reads in the swapped phase, then in it again after the natural one
        big.step(steps)
        small.step(steps)
        _assert_repeats(big, small, 0)
    assert big.residual().nonfinite == 0


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("scheme", [capi.LBM_SCHEME_TWO_PASS, capi.LBM_SCHEME_LAGGED])
def test_large_runs_with_wet_nodes_repeat_small_ones(storage, scheme):
    w = workloads.wet_box(D=3, n=(60, 40, 16), faces={"x-": "inlet", "x+": "pressure",
                                                      "z-": "periodic", "z+": "periodic"})
    kw = dict(storage=STORAGE[storage], scheme=scheme)
    big = capi.Solver.from_workload(_repeated(w, 0, _times(w, storage)), **kw)
    small = capi.Solver.from_workload(w, **kw)
    big.step(3)
    small.step(3)
    _assert_repeats(big, small, 0)


@pytest.mark.parametrize("solids", [False, True])
@pytest.mark.parametrize("scheme", [capi.LBM_SCHEME_TWO_PASS, capi.LBM_SCHEME_LAGGED])
@pytest.mark.parametrize("storage,nx", [("f64", 70), ("f32", 70), ("f32", 64), ("f16", 70),
                                        ("bf16", 64)])
def test_large_rounds_of_the_server(storage, nx, scheme, solids):
    """A round whose runs together exceed the cache: a large run, a small one of the same group and
    one stepped by launches of its own, each against the same run alone."""
    w = _base(nx, solids)
    wet = workloads.wet_box(D=3, n=(30, 20, 10))
    kw = dict(storage=STORAGE[storage], scheme=scheme)
    srv = capi.Server(pool_bytes=3 << 30, check_every=4)
    big, small, solo = [srv.submit(x, shift=1, tol=1e-300, max_steps=10 ** 6, **kw)
                        for x in (_repeated(w, 0, _times(w, storage)), w, wet)]
    srv.progress(1)
    for rid, x in ((small, w), (solo, wet)):
        alone = capi.Solver.from_workload(x, shift=1, **kw)
        alone.step(4)
        _assert_repeats(srv.solver(rid), alone, 0)
    _assert_repeats(srv.solver(big), srv.solver(small), 0)
    srv.close()
