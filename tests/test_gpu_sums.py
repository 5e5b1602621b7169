"""Passes that only sum: the ensemble's mass and energy (one reading pass per axis for all runs
of a size), the power sums of the structure functions, and the vortex-ring generator's brick
and profile products, at the sizes where their tiles and bricks have remainders."""
import numpy as np
import pytest

import gp_inputs as I
from oracle import gp as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_batch_energies_match_single_plans(prec):
    """Ragged and one-axis shapes, groups of one and of several runs, before and after the
    step graphs know the states, and with states they do not know.  Both sides sum the
    same transforms in FP64, in another order: 1e-12."""
    import paper_2003_03590_amd as gp
    shapes = [(16, 16, 16), (96, 3, 8), (16, 16, 16), (1, 24, 1), (2, 48, 12), (16, 16, 16), (64, 64, 1)]
    par = [dict(n=s, alpha=0.2 + 0.1 * i, beta=3.0 + i, dt=0.01) for i, s in enumerate(shapes)]
    bp = gp.BatchPlan(par, prec)
    plans = [gp.Plan(q["n"], q["alpha"], q["beta"], q["dt"], prec) for q in par]
    mk = lambda seed: [torch.from_numpy(I.random_field(s[::-1], seed=seed + i)).to(DEV).to(bp.dtype).contiguous()
                       for i, s in enumerate(shapes)]
    known, other = mk(10), mk(50)
    for states in (known, bp.step_n(known, 2), other, known):
        got = bp.energies(states)
        for i, (p, s) in enumerate(zip(plans, states)):
            e = p.energies(s)
            assert abs(got[i, 0] - e["mass"]) <= 1e-12 * e["mass"], (i, shapes[i])
            assert abs(got[i, 1] - e["energy"]) <= 1e-12 * e["energy"], (i, shapes[i])


def test_batch_energies_not_finite():
    import paper_2003_03590_amd as gp
    from paper_2003_03590_amd import _lib as L
    bp = gp.BatchPlan([dict(n=16, alpha=0.2, beta=3.0, dt=0.01)] * 2, "c128")
    states = [torch.ones((16, 16, 16), dtype=torch.complex128, device=DEV) for _ in range(2)]
    states[1][3, 2, 1] = float("nan")
    with pytest.raises(gp.GPError) as ei:
        bp.energies(states)
    assert ei.value.status == L.GP_ERR_NONFINITE
    states[1][3, 2, 1] = 1.0
    assert np.allclose(bp.energies(states)[:, 0], 1.0, rtol=1e-13)


@pytest.mark.parametrize("n", [2, 3, 6, 16, 24, 32, 48, 64, 96])
@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_structure_functions_of_every_tile(n, prec):
    """One-stage schedules (no exchange buffer of their own), tiles wider than the grid, and
    every compiled variant of the length; FP64 transforms round by 1e-15 a stage, FP32 ones by
    1e-7, relative to the field's power."""
    import paper_2003_03590_amd as gp
    alpha = 0.3
    plan = gp.Plan(n, alpha, 3.0, 0.01, prec)
    psi = np.exp(0.3 * I.random_real((n,) * 3, 7)) * np.exp(0.5j * I.random_real((n,) * 3, 8))
    psi = psi.astype(np.complex64 if prec == "c64" else np.complex128)
    t = torch.from_numpy(psi).to(DEV)
    ref = O.structure_function_density(psi.astype(np.complex128))
    vref, v2ref = O.structure_function_velocity(psi.astype(np.complex128), alpha)
    tol = 1e-12 if prec == "c128" else 2e-5
    for v in range(gp.lib().gp_variant_count(n, plan.prec)):
        for a in range(3):
            plan.select_variant(a, v)
        got = plan.structure_fn(t)
        vel, v2 = plan.structure_fn_velocity(t)
        assert np.max(np.abs(got - ref)) <= tol * np.max(ref), (n, prec, v)
        assert np.max(np.abs(vel - vref)) <= tol * np.max(v2ref), (n, prec, v)
        assert np.max(np.abs(v2 - v2ref)) <= tol * np.max(v2ref), (n, prec, v)
    plan.close()


@pytest.mark.parametrize("shape", [(8, 8, 8), (12, 24, 2), (1, 3, 16), (32, 6, 4)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("far", [False, True], ids=["near", "far"])
def test_vortex_rings_in_bricks(shape, far):
    """Bricks past the grid's end, all permutations, translations outside [0, 2 pi), and lengths
    beyond which every image takes its own root.  An image's factor rounds by a few units in the
    last place of its coordinates (far: of a length of 200): 42 factors, 2e-13 (far: 1e-11)."""
    import paper_2003_03590_amd as gp
    nx, ny, nz = shape
    plan = gp.Plan(shape, 0.1, 20.0, 1e-3, "c128")
    rng = np.random.default_rng(5)
    xi = 0.07
    R = 150.0 if far else 0.5
    pairs = [(R + 0.1 * q, 2.0 * R + 0.3 * q, *rng.uniform(-7.0, 13.0, 3), q) for q in range(6)]
    got = plan.init_rvr(pairs, xi).cpu().numpy()
    c = [2 * np.pi * np.arange(m) / m for m in shape]
    coords = (c[0][None, None, :], c[1][None, :, None], c[2][:, None, None])
    ref = np.ones((nz, ny, nx), dtype=np.complex128)
    for r, d, X, Y, Z, perm in pairs:
        a = [coords[i] for i in I.PERMUTATIONS[perm]]
        s = np.broadcast_arrays(*(np.mod(u - t, 2 * np.pi) for u, t in zip(a, (X, Y, Z))))
        ref = ref * I._pair_periodic(*s, r, d, xi)
    assert np.max(np.abs(got - ref)) <= (1e-11 if far else 2e-13)
    plan.close()


@pytest.mark.parametrize("shape", [(96, 3, 6), (6, 48, 12), (3, 2, 24), (64, 12, 8)])
@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_helicity_at_tile_remainders(shape, prec):
    """The Hessian passes with a last tile of few pencils, odd extents (mirror pairs without a
    Nyquist plane) and short axes.  Tolerances as for the sizes with whole tiles: round-off
    amplified by the divisions by |psi|^2 and |grad psi|^2 near cores and stagnation points."""
    import paper_2003_03590_amd as gp
    from oracle import helicity as OH
    psi = I.random_field(shape[::-1], seed=71)
    base = psi.astype(np.complex64).astype(np.complex128) if prec == "c64" else psi
    ref = OH.helicity(base, 0.3)
    v, om = O.velocity(base, 0.3), OH.curl(O.velocity(base, 0.3))
    scale = float(np.mean(np.sqrt(sum(c * c for c in v)) * np.sqrt(sum(c * c for c in om))))
    plan = gp.Plan(shape, 0.3, 2.0, 1e-3, prec)
    H, Hreg, spec = plan.helicity(torch.from_numpy(psi).to(DEV).to(plan.dtype).contiguous())
    tol = 1e-10 if prec == "c128" else 1e-3
    assert abs(H - ref["H"]) < tol * scale and abs(Hreg - ref["H_reg"]) < tol * scale
    assert np.abs(spec - ref["spec"]).max() < tol * scale
    plan.close()
