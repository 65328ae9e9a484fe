"""Device memory of a solver that steps in one launch from one population buffer into a second."""
import pytest

from paper_2606_29619_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
capi = pytest.importorskip("paper_2606_29619_amd.capi")


def test_workspace_that_does_not_fit_with_a_second_buffer(monkeypatch):
    """Where memory for the second population buffer is not there, a solver is made without it."""
    w = workloads.random_porosity_2d(nx=130, ny=64, seed=6, ell=3.0, nu=0.03, b=2e-4)
    a = capi.Solver.from_workload(w, storage=capi.LBM_F32)
    b = capi.Solver.from_workload(w, storage=capi.LBM_F32, passes=capi.LBM_PASSES_SEPARATE)
    empty = torch.empty

    def small_memory(*size, **kw):
        if kw.get("dtype") == torch.uint8 and size[0] > b.nbytes:
            raise torch.cuda.OutOfMemoryError("not enough memory")
        return empty(*size, **kw)

    monkeypatch.setattr(torch, "empty", small_memory)
    c = capi.Solver.from_workload(w, storage=capi.LBM_F32)
    with pytest.raises(torch.cuda.OutOfMemoryError):  # nothing smaller to fall back to
        capi.Solver.from_workload(w, storage=capi.LBM_F64, scheme=capi.LBM_SCHEME_LAGGED)
    monkeypatch.undo()
    assert a.nbytes > b.nbytes == c.nbytes
    a.step(5)
    assert c.step_timed(1)[0] > 0.0
    c.step(4)
    assert torch.equal(a.populations(), c.populations())
