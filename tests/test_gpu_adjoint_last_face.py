"""The last face of a segment in the adjoint along lines of full chunks (16 cells), halved ones,
one cell more or less, and uneven segments, against reverse-mode AD of the PyTorch restatement
of the oracle.  Tolerance as for the other line lengths: 1e3 rounded terms per point times 1e2
from the weights times 1e-16 = 1e-11 of the largest component."""
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


@pytest.mark.parametrize("shape,weno", [((16, 16, 16), "js"), ((17, 15, 32), "z"), ((48, 12, 31), "m"), ((8, 33, 47), "js"),
                                        ((32, 64, 48), "js")])
def test_last_faces(orc, shape, weno):
    print(f"[case] adjoint last face {shape} weno-{weno}", flush=True)
    rho, vel, p, _ = I.smooth_primitives(shape, seed=9, amp=0.3, kmax=3)
    rng = np.random.default_rng(9)
    rho, p = (q * (1.0 + 0.05 * rng.standard_normal(shape)) for q in (rho, p))
    rbar = rng.standard_normal((5,) + shape)
    plan = Plan(shape, mu_eff=0.0, weno=weno)
    u, r = plan.init_state(rho, vel, p), torch.from_numpy(rbar).cuda()
    got = plan.rhs_vjp(u, r)
    ref = tr.rhs_vjp(torch.from_numpy(orc.init_state(rho, vel, p)), torch.from_numpy(rbar),
                     tr.make_phys(mu=0.0, delta=1e-6, weights=weno)).numpy()
    assert rel_max(got.cpu().numpy(), ref) <= 1e-11
    assert torch.equal(plan.rhs_vjp(u, r), got)  # the same bits every time
