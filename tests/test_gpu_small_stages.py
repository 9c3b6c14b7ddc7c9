"""Small boxes run a stage's kernels side by side and sum them point by point; larger ones
(and other launch shapes) one after the other.  The sums take the same terms in the same order
with the same roundings, so the two have to agree bit for bit.  Also the x rows at the row
lengths where that kernel changes (two cells per thread, odd rows, chunks past 512), against
the oracle at the bound of the parity tests (1e-12 per evaluation)."""
import numpy as np
import pytest

from conftest import rel_max
from paper_2211_16718_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2211_16718_amd.api import Ensemble, Plan  # noqa: E402


def prims(shape, seed=5):
    rho, vel, p, _ = I.smooth_primitives(shape, seed=seed, amp=0.3, kmax=3)
    rng = np.random.default_rng(seed)
    return rho * (1.0 + 0.05 * rng.standard_normal(shape)), vel, p * (1.0 + 0.05 * rng.standard_normal(shape))


@pytest.mark.parametrize("shape", [(8, 8, 8), (9, 17, 31), (20, 9, 66), (8, 8, 512), (33, 40, 70), (72, 70, 74)])
@pytest.mark.parametrize("mu,weno", [(0.02, "js"), (0.02, "z"), (0.0, "m")])
def test_side_by_side_and_in_turn_agree_bitwise(shape, mu, weno):
    print(f"[case] small stages {shape} mu={mu} weno-{weno}", flush=True)
    a, b = Plan(shape, mu_eff=mu, weno=weno), Plan(shape, mu_eff=mu, weno=weno)
    b.set_tiles(block=128)  # in turn
    u = a.init_state(*prims(shape))
    assert torch.equal(a.rhs(u), b.rhs(u))
    for step in ("rk4", "tvdrk3"):
        ua, ub = u.clone(), u.clone()
        da, db = getattr(a, step)(ua, 1e-4, 3), getattr(b, step)(ub, 1e-4, 3)
        assert torch.equal(ua, ub)
        assert torch.equal(da, db)
    # the checkpointed forward keeps its stage states outside the plan's buffers
    ja, ga = a.adjoint_rk4(u, 1e-4, 3, 2)
    jb, gb = b.adjoint_rk4(u, 1e-4, 3, 2)
    assert torch.equal(ja, jb) and torch.equal(ga, gb)


@pytest.mark.parametrize("graph", [False, True])
def test_small_ensemble_equals_its_boxes(graph):
    print(f"[case] small ensemble graph={graph}", flush=True)
    stream = torch.cuda.Stream()
    boxes = [dict(shape=s, mu_eff=0.02, dt=1e-4 * (i + 1)) for i, s in enumerate([(8, 12, 16), (20, 9, 33), (31, 8, 40)])]
    ens = Ensemble(boxes, stream=stream)
    with torch.cuda.stream(stream):
        plans = [Plan(b["shape"], mu_eff=b["mu_eff"], stream=stream) for b in boxes]
        states = [plan.init_state(*prims(b["shape"], i), out=ens.state(i)).clone()
                  for i, (plan, b) in enumerate(zip(plans, boxes))]
        for _ in range(3):  # replays after the first round of the graph
            ens.run(2, diag=True, graph=graph)
            for i, (plan, u) in enumerate(zip(plans, states)):
                plan.rk4(u, boxes[i]["dt"], 2)
                stream.synchronize()
                assert torch.equal(ens.state(i), u)


@pytest.mark.parametrize("shape", [(8, 9, 255), (8, 8, 256), (9, 8, 257), (8, 8, 511), (8, 8, 513), (8, 9, 1025), (8, 8, 1536)])
def test_row_lengths_match_oracle(orc, shape):
    print(f"[case] x rows {shape}", flush=True)
    rho, vel, p = prims(shape)
    plan = Plan(shape, mu_eff=0.01)
    u = plan.init_state(rho, vel, p)
    ref = orc.rhs(orc.init_state(rho, vel, p), orc.make_phys(mu_eff=0.01))
    assert rel_max(plan.rhs(u).cpu().numpy(), ref) <= 1e-12
