"""A record has the same bits whichever kernel forms it: the diagnostics kernel in either of its
variants (by launched blocks), the wave speed alone and, while every tile has a partial sum of
its own (up to 1024 tiles), the viscous kernel of the next step.  All sum the same point
quantities over the same tiles in the same order; above 1024 tiles a block of the diagnostics
kernel sums several tiles before its threads', the viscous kernel each tile by itself."""
import pytest

from paper_2211_16718_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2211_16718_amd.api import Ensemble, Plan  # noqa: E402


def prims(shape):
    return I.smooth_primitives(shape, seed=11, amp=0.3, kmax=3)[:3]


def test_record_does_not_depend_on_the_launched_blocks():
    print("[case] records by launched blocks", flush=True)
    shape = (64, 128, 128)  # 1024 tiles of four planes
    got = []
    for tile_grid in (0, 1000, 768, 300):
        ens = Ensemble([dict(shape=shape, mu_eff=0.0, dt=1e-4)])
        ens.set_launch(tile_grid=tile_grid)
        Plan(shape, mu_eff=0.0).init_state(*prims(shape), out=ens.state(0))
        got.append(ens.run(2, diag=True, graph=False))
        torch.cuda.synchronize()
    assert all(torch.equal(got[0], d) for d in got[1:])


@pytest.mark.parametrize("shape,tiles", [((17, 20, 33), 54), ((64, 64, 64), 256), ((128, 96, 100), 1536)])
@pytest.mark.parametrize("block", [0, 128])  # side by side where small, in turn
def test_record_of_the_viscous_kernel_is_that_of_the_diagnostics_kernel(shape, tiles, block):
    print(f"[case] fused records {shape} block={block}", flush=True)
    plan = Plan(shape, mu_eff=0.02)
    plan.set_tiles(block=block)
    u = plan.init_state(*prims(shape))
    v = u.clone()
    d = plan.rk4(u, 1e-4, 3)  # the first two by the next step's viscous kernel
    one = torch.cat([plan.rk4(v, 1e-4, 1) for _ in range(3)])
    assert torch.equal(u, v)
    assert torch.equal(d[2], one[2])
    assert tiles > 1024 or torch.equal(d, one)
    assert torch.equal(plan.diagnostics(u), d[2])
    assert torch.equal(plan.max_wave_speed(u)[0], d[2, 7])
