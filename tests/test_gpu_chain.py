"""How the passes of a step are cut does not change a state: the arithmetic of a sub-step is
written out (which products are fused), so the running chain, single sub-steps and the
ensemble's graphs give the same bits when they take the axes in the same order."""
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
