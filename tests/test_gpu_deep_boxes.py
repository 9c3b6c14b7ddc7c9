"""Boxes of 256 and more planes with few columns, whose blocks of the viscous and diagnostics
kernels take as few planes as those of other small boxes, and the viscous terms alone, which
choose their planes for a launch of their own: against the oracle at the bound of the parity
tests (1e-12 per evaluation), and the stage's launches side by side against in turn."""
import numpy as np
import pytest

from conftest import rel_max
from paper_2211_16718_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2211_16718_amd.api import Plan  # noqa: E402


@pytest.mark.parametrize("shape", [(256, 8, 8), (257, 9, 11), (300, 16, 40), (270, 33, 65), (256, 64, 64)])
def test_deep_boxes(orc, shape):
    print(f"[case] deep box {shape}", flush=True)
    rho, vel, p, _ = I.smooth_primitives(shape, seed=2, amp=0.3, kmax=3)
    rng = np.random.default_rng(2)
    rho, p = (q * (1.0 + 0.05 * rng.standard_normal(shape)) for q in (rho, p))
    u0, ph = orc.init_state(rho, vel, p), orc.make_phys(mu_eff=0.02)
    a, b = Plan(shape, mu_eff=0.02), Plan(shape, mu_eff=0.02)
    b.set_tiles(block=128)  # in turn
    u = a.init_state(rho, vel, p)
    assert rel_max(a.viscous(u).cpu().numpy(), orc.viscous(u0, ph)) <= 1e-12
    assert rel_max(a.rhs(u).cpu().numpy(), orc.rhs(u0, ph)) <= 1e-12
    assert rel_max(a.diagnostics(u).cpu().numpy(), orc.diag(u0, ph)) <= 1e-12
    assert torch.equal(a.viscous(u), b.viscous(u))
    v = u.clone()
    da, db = a.rk4(u, 1e-4, 3), b.rk4(v, 1e-4, 3)
    assert torch.equal(u, v) and torch.equal(da, db)


@pytest.mark.parametrize("shape", [(128, 128, 8), (9, 8, 8), (40, 70, 33), (66, 90, 130)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_viscous_terms_alone(orc, shape, precision):
    print(f"[case] viscous terms {shape} {precision}", flush=True)
    rho, vel, p, _ = I.smooth_primitives(shape, seed=3, amp=0.3, kmax=3)
    plan = Plan(shape, mu_eff=0.02, precision=precision)
    got = plan.viscous(plan.init_state(rho, vel, p)).double().cpu().numpy()
    # FP32 state: 24 bits, amplified by two derivatives of spacing h (1/h^2 against fields of wavenumber 3)
    tol = 1e-12 if precision == "fp64" else 6e-8 * 16 * (max(shape) / 3.0) ** 2
    assert rel_max(got, orc.viscous(orc.init_state(rho, vel, p), orc.make_phys(mu_eff=0.02))) <= tol
