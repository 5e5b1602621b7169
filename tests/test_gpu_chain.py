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


def _forced(shape, prec, coef, choice, path):
    """A plan whose chain was chosen by a tuning file: choice = carrier + 3 for the plain form."""
    import json

    import paper_2003_03590_amd as gp
    plan = gp.Plan(shape, 0.3, coef / 0.01, 0.01, prec)
    plan.select_variant(4, choice % 3)           # ends a plane pass that is on by default
    key = "{}/{}/{}x{}x{}/t2/a".format(torch.cuda.get_device_properties(0).gcnArchName.split(":")[0], prec, *shape)
    path.write_text(json.dumps({key + "0": 0, key + "1": 0, key + "2": 0, key + "3/r1": 0, key + "4": choice, key + "5": 0}))
    plan.autotune(reps=1, cache=str(path))
    assert plan.schedule(4) == "nl: " + "xyz"[choice % 3] + " pass" + (", plain" if choice > 2 else "")
    return plan


@pytest.mark.parametrize("coef", [0.04, 0.5], ids=["small", "mixed"])
@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("shape", [(96, 48, 24), (24, 192, 2), (48, 16, 128), (384, 8, 6), (6, 384, 768), (768, 12, 384),
                                   (1, 64, 12)], ids=lambda s: "x".join(map(str, s)))
def test_steps_are_bitwise_their_substeps(shape, prec, coef, tmp_path):
    """The chain x y z N z y x N ... against single sub-steps: a turning pass equals the two
    passes and the rotation that it replaces, and the plain form takes these.  Every carrier,
    both forms, one to three steps; 384 and 768 points along each axis."""
    psi0 = _state(shape, prec, 51)
    for choice in range(6):
        first = choice % 3
        if shape[first] == 1:
            continue
        plan = _forced(shape, prec, coef, choice, tmp_path / "tune.json")
        order = [first, 1 if first == 0 else 0, 1 if first == 2 else 2]
        for n in (1, 2, 3):
            a = plan.step_n(psi0.clone(), n)
            b = psi0.clone()
            for k in range(n + 1):
                if k:
                    plan.substep_nonlinear(b, 0.01)
                for axis in (order[::-1] if k % 2 else order):
                    plan.substep_linear(b, axis, 0.005 if k in (0, n) else 0.01)
            assert _same(a, b), (choice, n)
        plan.close()


@pytest.mark.parametrize("shape,prec", [((384, 12, 6), "c128"), ((12, 384, 384), "c128"), ((192, 24, 384), "c128"),
                                        ((384, 96, 24), "c128"), ((768, 384, 8), "c128"), ((384, 768, 1), "c128"),
                                        ((1, 24, 384), "c128"), ((192, 8, 6), "c64"), ((1024, 6, 4), "c64"),
                                        ((512, 12, 8), "c64"), ((384, 8, 6), "c64")],
                         ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_default_chain_on_long_axes(shape, prec):
    """Shapes at which the default takes another first axis or the plain form, against the
    oracle's literal steps (round-off of three steps)."""
    import paper_2003_03590_amd as gp
    from oracle import gp as O
    psi0 = I.random_field(shape[::-1], seed=35)
    base = psi0.astype(np.complex64).astype(np.complex128) if prec == "c64" else psi0
    plan = gp.Plan(shape, 0.3, 4.0, 0.01, prec)
    for n in (3, -2):
        got = plan.step_n(torch.from_numpy(psi0).to(DEV).to(plan.dtype).contiguous(), n).cpu().numpy()
        ref = O.evolve(base, 0.3, 4.0, 0.01, n)
        assert np.linalg.norm(got - ref) < (1e-12 if prec == "c128" else 5e-6) * np.linalg.norm(ref)
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


def test_tuning_file_of_three_passes_a_step_is_not_obeyed(tmp_path):
    """Entries without the tag of the running chain were timed for another one: a file that holds
    only such entries is timed again and keeps them."""
    import json

    import paper_2003_03590_amd as gp
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    old = {f"{arch}/c64/128x128x128/a{a}": v for a, v in enumerate((2, 2, 2))}
    old[f"{arch}/c64/128x128x128/a4"] = 2
    path = tmp_path / "tune.json"
    path.write_text(json.dumps(old))
    plan = gp.Plan(128, 0.3, 4.0, 0.01, "c64")
    plan.autotune(reps=2, cache=str(path))
    data = json.loads(path.read_text())
    assert all(data[k] == v for k, v in old.items())
    assert {k.split("/")[-1] for k in data if "/t2/" in k} >= {"a0", "a1", "a2", "a4"}
    assert plan.schedule(4) != "nl: z pass"          # z is never timed as the first axis
    plan.close()


def test_tuning_starts_from_a_state_of_its_own():
    """The time of a turning pass depends on the angles: what the caller's scratch state holds
    does not count."""
    import ctypes as C

    import paper_2003_03590_amd as gp
    plan = gp.Plan((128, 2, 2), 0.3, 4.0, 0.01, "c64")
    scratch = torch.full(plan.shape, float("nan"), dtype=plan.dtype, device=DEV)
    bp = gp.BatchPlan([dict(n=(128, 2, 2), alpha=0.3, beta=4.0, dt=0.01)], "c64")
    assert gp.lib().gp_autotune(bp._h, C.c_void_p(scratch.data_ptr()), 2, None) == 0
    torch.cuda.synchronize()
    assert bool(torch.isfinite(torch.view_as_real(scratch)).all())
    plan.close()
    bp.close()


@pytest.mark.parametrize("coef", [0.04, 0.5], ids=["small", "mixed"])
@pytest.mark.parametrize("shape", [(96, 48, 24), (24, 64, 1), (1, 48, 1), (192, 6, 4), (4, 384, 6), (2, 6, 768)],
                         ids=lambda s: "x".join(map(str, s)))
def test_adjoint_on_axes_of_several_stages(shape, coef):
    """The passes that store the tape and those that rotate by it, along axes whose schedules have
    two and three stages, against the oracle; one, two and three real axes.  The bound is 1e-12, a
    few hundred times one step's round-off, times the growth of an error through n adjoint
    rotations, each of which multiplies by up to 1 + 2 coef |phi|^2 (|phi|^2 of about 2)."""
    import paper_2003_03590_amd as gp
    from oracle import adjoint as OA
    alpha, dt = 0.3, 0.01
    beta = coef / dt
    psi0, lam0 = I.random_field(shape[::-1], seed=61), I.random_field(shape[::-1], seed=62)
    plan = gp.Plan(shape, alpha, beta, dt, "c128")
    for n in (1, 2, 5):
        lam = torch.from_numpy(lam0).to(DEV)
        plan.adjoint_step_n(torch.from_numpy(psi0).to(DEV), lam, n)
        states, ref = OA.forward_states(psi0, alpha, beta, dt, n), lam0
        for k in range(n - 1, -1, -1):
            ref = OA.step_adjoint(states[k], ref, alpha, beta, dt)
        err = np.linalg.norm(lam.cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err < 1e-12 * (1 + 4 * coef) ** n, n
    plan.close()
