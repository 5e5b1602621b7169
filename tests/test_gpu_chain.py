"""How the passes of a step are cut does not change a state: the arithmetic of a sub-step is
written out (which products are fused), so the running chain, single sub-steps and the
ensemble's graphs give the same bits when they take the axes in the same order."""
import numpy as np
import pytest

import gp_inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"


def _state(shape, prec, seed):
    dt = torch.complex128 if prec == "c128" else torch.complex64
    return torch.from_numpy(I.random_field(shape[::-1], seed=seed)).to(DEV).to(dt).contiguous()


def _same(a, b):
    return torch.equal(torch.view_as_real(a), torch.view_as_real(b))


@pytest.mark.parametrize("coef", [0.04, 0.5], ids=["small", "mixed"])
@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("shape", [(96, 48, 24), (24, 192, 2), (48, 16, 128), (384, 8, 6), (1, 64, 12)],
                         ids=lambda s: "x".join(map(str, s)))
def test_step_is_bitwise_its_substeps(shape, prec, coef):
    """One step (x y z N z y x) against single sub-steps: the turning pass equals the two
    passes and the rotation that it replaces."""
    import paper_2003_03590_amd as gp
    plan = gp.Plan(shape, 0.3, coef / 0.01, 0.01, prec)
    psi0 = _state(shape, prec, 51)
    a = plan.step_n(psi0.clone(), 1)
    b = psi0.clone()
    for axis in (0, 1, 2):
        plan.substep_linear(b, axis, 0.005)
    plan.substep_nonlinear(b, 0.01)
    for axis in (2, 1, 0):
        plan.substep_linear(b, axis, 0.005)
    assert _same(a, b)
    plan.close()


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_ensemble_run_is_bitwise_a_single_plan(prec):
    """Ensemble graphs (three size groups; even and odd counts, backward) against single plans
    with separate passes."""
    import paper_2003_03590_amd as gp
    runs = [dict(n=48, alpha=0.2, beta=3.0, dt=0.01), dict(n=96, alpha=0.1, beta=20.0, dt=1e-3),
            dict(n=48, alpha=0.3, beta=2.0, dt=0.01), dict(n=24, alpha=0.3, beta=50.0, dt=0.01)]
    bp = gp.BatchPlan(runs, prec)
    states = [_state((r["n"],) * 3, prec, 60 + i) for i, r in enumerate(runs)]
    refs = [s.clone() for s in states]
    plans = [gp.Plan(r["n"], r["alpha"], r["beta"], r["dt"], prec) for r in runs]
    for p in plans:
        p.select_variant(3, 0)
    for n in (1, 2, 3, 8, -6):
        bp.step_n(states, n)
        for p, r in zip(plans, refs):
            p.step_n(r, n)
        torch.cuda.synchronize()
        assert all(_same(s, r) for s, r in zip(states, refs)), n
    for p in plans:
        p.close()
    bp.close()


@pytest.mark.parametrize("lo,hi", [(0.0, 0.0625), (0.0625, 0.125), (0.1249, 0.1251), (0.125, 0.25)])
def test_rotation_across_the_border_of_the_short_series(lo, hi):
    """exp(-i beta (|psi|^2 - 1) dt) psi at angles around 1/16 and 1/8, both signs, beta dt = 1, in
    complex64, where FP64 is an exact reference.  A point is rounded once per component and its angle by |psi|^2 times a few ulp: 8 ulp.  The
    norm's relative change averages to sqrt(2) ulp / sqrt(points) = 1.7e-10 where
    a truncated series would leave its own error at every point: 6 of those."""
    import paper_2003_03590_amd as gp
    n = 64
    rng = np.random.default_rng(7)
    a = rng.uniform(lo, hi, (n, n, n)) * rng.choice([-1.0, 1.0], (n, n, n))
    psi0 = np.sqrt(1.0 - a) * np.exp(1j * rng.uniform(0.0, 2.0 * np.pi, (n, n, n)))
    plan = gp.Plan(n, 0.3, 100.0, 0.01, "c64")
    x = torch.from_numpy(psi0).to(DEV).to(plan.dtype).contiguous()
    x0 = x.cpu().numpy().astype(np.complex128)
    got = plan.substep_nonlinear(x, 0.01).cpu().numpy().astype(np.complex128)
    ref = x0 * np.exp(-1j * (np.abs(x0) ** 2 - 1.0))
    ulp = 2.0 ** -24
    assert np.abs(got - ref).max() < 8 * ulp
    assert abs(np.mean((np.abs(got) / np.abs(x0)) ** 2 - 1.0)) < 6 * np.sqrt(2.0) * ulp / n ** 1.5
    plan.close()
