"""The convective adjoint at the line lengths, counts and segment splits where it changes, for
every set of weights, against reverse-mode AD of the PyTorch restatement of the oracle.

Tolerance: the products sum some 1e3 rounded terms per point, and the WENO weights multiply
relative errors of the small indicators by up to 1e2, so 1e3 * 1e2 * 1e-16 = 1e-11 of the
largest component.
"""
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


@pytest.mark.parametrize("shape,weno", [  # (nz, ny, nx)
    ((9, 9, 9), "z"),       # two segments of 4 and 5 cells
    ((13, 17, 40), "m"),    # uneven segments, line counts that are no multiple of a block's
    ((41, 8, 33), "js"),
    ((8, 100, 24), "z"),    # many short segments
    ((8, 8, 63), "m"),      # x: one cell short of, exactly, and one cell past a chunk
    ((9, 8, 64), "js"),
    ((8, 9, 65), "z"),
    ((8, 8, 129), "m"),
    ((90, 70, 37), "js"),   # x: whole lines in three chunks; y, z: lanes
    ((66, 64, 65), "z"),    # y, z: the march
])
def test_rhs_vjp_lines(orc, shape, weno):
    print(f"[case] rhs_vjp lines {shape} weno-{weno}", flush=True)
    rho, vel, p, _ = I.smooth_primitives(shape, seed=5, amp=0.3, kmax=3)
    rng = np.random.default_rng(sum(shape))
    rho = rho * (1.0 + 0.05 * rng.standard_normal(shape))
    p = p * (1.0 + 0.05 * rng.standard_normal(shape))
    vel = vel + 0.1 * rng.standard_normal(vel.shape)
    mu = 0.02 if shape[2] % 2 else 0.0  # viscous boxes of 2, 4 and 8 planes per block
    plan = Plan(shape, mu_eff=mu, weno=weno)
    u = plan.init_state(rho, vel, p)
    rbar = rng.standard_normal((5,) + shape)
    r = torch.from_numpy(rbar).cuda()
    got = plan.rhs_vjp(u, r)
    ref = tr.rhs_vjp(torch.from_numpy(orc.init_state(rho, vel, p)), torch.from_numpy(rbar),
                     tr.make_phys(mu=mu, delta=1e-6, weights=weno)).numpy()
    assert rel_max(got.cpu().numpy(), ref) <= 1e-11
    assert torch.equal(plan.rhs_vjp(u, r), got)  # the same bits every time
