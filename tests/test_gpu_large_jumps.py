"""Jumps of a size that products of eight indicator factors do not represent: the mapped weights'
right-hand side (products of four) and the Jiang-Shu product of the adjoint (of seven), at the
bounds of the parity tests (1e-12 per evaluation, 1e-11 per product).  A velocity scale a, a
power of two, makes the rows (density, momentum, energy) of the state scale with 1, a, a^2 and
those of the right-hand side with a, a^2, a^3; rows are compared with these factors taken out."""
import numpy as np
import pytest

from conftest import rel_max
from paper_2211_16718_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle import torch_ref as tr  # noqa: E402
from paper_2211_16718_amd.api import Plan  # noqa: E402


def prims(shape, a):
    rho, vel, p, _ = I.smooth_primitives(shape, seed=7, amp=0.3, kmax=3)
    rng = np.random.default_rng(7)
    rho, p = (q * (1.0 + 0.05 * rng.standard_normal(shape)) for q in (rho, p))
    return rho, a * vel, a * a * p


def rows(x, s0, a):
    """x with row scales s0 (1, a, a, a, a^2) taken out."""
    return x / (s0 * np.array([1.0, a, a, a, a * a])).reshape(5, 1, 1, 1)


@pytest.mark.parametrize("shape", [(10, 12, 37), (8, 8, 520)])  # side by side with odd rows; in turn with chunked rows
def test_mapped_weights_at_large_jumps(orc, shape):
    print(f"[case] weno-m at large jumps {shape}", flush=True)
    a = 2.0 ** 27  # energy fluxes and their jumps of about 1e24: eight factors of their squares 1e384
    rho, vel, p = prims(shape, a)
    mu = 0.01 * a
    ref = orc.rhs(orc.init_state(rho, vel, p), orc.make_phys(mu_eff=mu, weno_weights=orc.WENO_M))
    assert np.isfinite(ref).all()
    plan = Plan(shape, mu_eff=mu, weno="m")
    got = plan.rhs(plan.init_state(rho, vel, p)).cpu().numpy()
    assert rel_max(rows(got, a, a), rows(ref, a, a)) <= 1e-12


@pytest.mark.parametrize("shape", [(10, 12, 37), (66, 64, 65)])  # a lane per cell; the march
def test_jiang_shu_product_at_large_jumps(orc, shape):
    print(f"[case] weno-js product at large jumps {shape}", flush=True)
    a = 2.0 ** 22
    rho, vel, p = prims(shape, a)
    u0 = orc.init_state(rho, vel, p)
    rbar = rows(np.random.default_rng(1).standard_normal((5,) + shape), a, a)
    ref = tr.rhs_vjp(torch.from_numpy(u0), torch.from_numpy(rbar), tr.make_phys(mu=0.01 * a, delta=1e-6)).numpy()
    assert np.isfinite(ref).all()
    plan = Plan(shape, mu_eff=0.01 * a)
    got = plan.rhs_vjp(plan.init_state(rho, vel, p), torch.from_numpy(rbar).cuda()).cpu().numpy()
    assert rel_max(rows(got, 1.0, 1.0 / a), rows(ref, 1.0, 1.0 / a)) <= 1e-11


@pytest.mark.parametrize("shape", [(10, 12, 37), (66, 64, 65)])
def test_weno_z_product_at_large_jumps(orc, shape):
    """The WENO-Z product forms no products of indicator factors, so jumps of the state beyond
    products of six (1e26) are in its range, also at the ends of segments, whose right-biased
    values are formed apart."""
    print(f"[case] weno-z product at large jumps {shape}", flush=True)
    a = 2.0 ** 44
    rho, vel, p = prims(shape, a)
    rbar = rows(np.random.default_rng(1).standard_normal((5,) + shape), a, a)
    ref = tr.rhs_vjp(torch.from_numpy(orc.init_state(rho, vel, p)), torch.from_numpy(rbar),
                     tr.make_phys(mu=0.01 * a, delta=1e-6, weights="z")).numpy()
    assert np.isfinite(ref).all()
    plan = Plan(shape, mu_eff=0.01 * a, weno="z")
    got = plan.rhs_vjp(plan.init_state(rho, vel, p), torch.from_numpy(rbar).cuda()).cpu().numpy()
    assert rel_max(rows(got, 1.0, 1.0 / a), rows(ref, 1.0, 1.0 / a)) <= 1e-11
