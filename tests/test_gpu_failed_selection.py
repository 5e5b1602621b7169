"""A selection or a tuning that finds no memory for its tables leaves the plan as it was: the same
schedules, the same bits of the next steps, and the selection can be made later; a call that
needs memory for itself leaves the plan usable.  (The failure
is forced on the host: every device allocation is refused before it is made.)"""
import pytest

import gp_inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"


def _state(shape, plan, seed=71):
    return torch.from_numpy(I.random_field(shape[::-1], seed=seed)).to(DEV).to(plan.dtype).contiguous()


def _same(a, b):
    return torch.equal(torch.view_as_real(a), torch.view_as_real(b))


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("shape,axis,variant", [((96, 8, 4), 0, 1), ((4, 128, 2), 1, 1), ((4, 2, 64), 2, 1),
                                                ((48, 48, 2), 3, 1), ((32, 32, 32), 5, 1), ((32, 32, 32), 5, 2)])
def test_failed_selection_changes_nothing(monkeypatch, shape, axis, variant, prec):
    import paper_2003_03590_amd as gp
    if axis == 3 and prec == "c64":            # 48 points start with the plane pass there
        shape = (96, 96, 2)
    plan = gp.Plan(shape, 0.3, 4.0, 0.01, prec)
    if axis != 3:
        plan.select_variant(4, 0)              # separate passes
    psi0 = _state(shape, plan)
    before = plan.step_n(psi0.clone(), 3)
    names = [plan.schedule(a) for a in range(6)]
    monkeypatch.setenv("GP_FAULT_INJECT", "alloc")
    for _ in range(2):
        with pytest.raises(gp.GPError) as ei:
            plan.select_variant(axis, variant)
        assert ei.value.status == gp._lib.GP_ERR_NOMEM
    monkeypatch.delenv("GP_FAULT_INJECT")
    assert [plan.schedule(a) for a in range(6)] == names
    assert _same(plan.step_n(psi0.clone(), 3), before)
    plan.select_variant(axis, variant)
    after = plan.step_n(psi0.clone(), 3)
    rel = float(torch.linalg.vector_norm(after - before) / torch.linalg.vector_norm(before))
    assert rel < (1e-13 if prec == "c128" else 3e-6)      # round-off of 10 passes
    plan.close()


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_failed_tuning_changes_nothing(monkeypatch, prec):
    import paper_2003_03590_amd as gp
    plan = gp.Plan((96, 64, 8), 0.3, 4.0, 0.01, prec)
    bp = gp.BatchPlan([dict(n=64, alpha=0.3, beta=4.0, dt=0.01), dict(n=24, alpha=0.2, beta=4.0, dt=0.01),
                       dict(n=64, alpha=0.2, beta=5.0, dt=0.01)], prec)
    psi0 = _state((96, 64, 8), plan)
    first = [_state((n,) * 3, plan, 80 + i) for i, n in enumerate((64, 24, 64))]
    one = plan.step_n(psi0.clone(), 3)
    many = bp.step_n([s.clone() for s in first], 3)
    monkeypatch.setenv("GP_FAULT_INJECT", "alloc")
    for p in (plan, bp):
        with pytest.raises(gp.GPError) as ei:
            p.autotune(reps=2)
        assert ei.value.status == gp._lib.GP_ERR_NOMEM
    monkeypatch.delenv("GP_FAULT_INJECT")
    assert _same(plan.step_n(psi0.clone(), 3), one)
    for n in (3, 4):       # a recorded length and one that records new graphs
        again = bp.step_n([s.clone() for s in first], n)
        ref = many if n == 3 else [s.clone() for s in first]
        if n == 4:
            fresh = gp.BatchPlan([dict(n=64, alpha=0.3, beta=4.0, dt=0.01), dict(n=24, alpha=0.2, beta=4.0, dt=0.01),
                                  dict(n=64, alpha=0.2, beta=5.0, dt=0.01)], prec)
            fresh.step_n(ref, 4)
            torch.cuda.synchronize()
            fresh.close()
        torch.cuda.synchronize()
        assert all(_same(a, b) for a, b in zip(again, ref))
    plan.close()
    bp.close()


def test_vortex_rings_without_memory(monkeypatch):
    """The pairs and their coordinates need device memory for the call."""
    import paper_2003_03590_amd as gp
    plan = gp.Plan((24, 16, 8), 0.3, 4.0, 0.01, "c128")
    pairs = [(1.5, 3.0, 1.0, 2.0, 3.0, 4), (1.0, 2.0, 4.0, 5.0, 0.5, 1)]
    ref = plan.init_rvr(pairs, 0.3)
    out = torch.full_like(ref, 7.0)
    monkeypatch.setenv("GP_FAULT_INJECT", "alloc")
    with pytest.raises(gp.GPError) as ei:
        plan.init_rvr(pairs, 0.3, out=out)
    assert ei.value.status == gp._lib.GP_ERR_NOMEM
    monkeypatch.delenv("GP_FAULT_INJECT")
    assert bool((out == 7.0).all())
    assert _same(plan.init_rvr(pairs, 0.3, out=out), ref)          # the plan is still usable
    plan.close()
