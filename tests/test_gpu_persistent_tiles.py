"""Launched blocks of the viscous kernel that take several virtual blocks each, of boxes whose
tile counts let the wave that holds a halo point change from one virtual block to the next.
Every virtual block computes the same whichever launched block runs it, so the results are
those of one launched block per virtual block, bit for bit."""
import bisect
import time

import numpy as np
import pytest

from paper_2211_16718_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2211_16718_amd.api import Ensemble, Plan  # noqa: E402

SHAPES = [(40, 44, 70), (33, 20, 100), (48, 64, 33)]  # nz, ny, nx


def owner_changes(grid, planes):
    """Consecutive virtual blocks of one launched block whose index within the box differs in
    bit 5, for tiles of 32 x 8 columns and `planes` planes (the blocks' walk in cns_batch.h)."""
    off = [0]
    for nz, ny, nx in SHAPES:
        off.append(off[-1] + -(-nx // 32) * -(-ny // 8) * -(-nz // planes))
    total, n = off[-1], 0
    xcds = min(grid, 8)
    for b in range(min(grid, total)):
        x, first = b % xcds, b // xcds
        q, r = divmod(total, xcds)
        lo = x * q + min(x, r)
        vbs = range(lo + first, lo + q + (x < r), grid // xcds + (x < grid % xcds))
        lbs = [v - off[bisect.bisect_right(off, v) - 1] for v in vbs]
        n += sum((i ^ j) & 32 != 0 for i, j in zip(lbs, lbs[1:]))
    return n


@pytest.mark.parametrize("grid", [3, 20, 40])
@pytest.mark.parametrize("diag", [False, True])
def test_looping_viscous_blocks_give_the_same_bits(grid, diag):
    print(f"[case] looping viscous blocks grid={grid} diag={diag}", flush=True)
    assert all(owner_changes(grid, planes) for planes in (4, 8, 16))
    stream = torch.cuda.Stream()
    out = []
    for tile_grid in (0, grid):
        ens = Ensemble([dict(shape=s, mu_eff=0.02, dt=1e-4) for s in SHAPES], stream=stream)
        ens.set_tiles(block=128)  # the kernels one after the other
        ens.set_launch(tile_grid=tile_grid)
        with torch.cuda.stream(stream):
            for i, s in enumerate(SHAPES):
                rho, vel, p, _ = I.smooth_primitives(s, seed=i, amp=0.3, kmax=3)
                noise = np.random.default_rng(i).standard_normal(s)
                Plan(s, mu_eff=0.02, stream=stream).init_state(rho * (1.0 + 0.05 * noise), vel, p, out=ens.state(i))
            d = ens.run(3, diag=diag, graph=False)
        stream.synchronize()
        out.append(([ens.state(i).clone() for i in range(len(SHAPES))], d))
    for a, b in zip(out[0][0], out[1][0]):
        assert torch.equal(a, b)
    if diag:
        assert torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("grids", [(1, 0), (0, 1), (1, 1)])
def test_launched_blocks_take_effect_in_a_small_batch(grids):
    """A 48^3 box (its stages side by side by default) with one launched block per kernel:
    one CU of 256 does the work of a sweep or of the viscous kernel, so a step takes many
    times as long, and gives the same bits."""
    print(f"[case] launched blocks {grids} of a small batch", flush=True)
    shape, stream = (48, 48, 48), torch.cuda.Stream()
    out, took = [], []
    for sweep_grid, tile_grid in ((0, 0), grids):
        ens = Ensemble([dict(shape=shape, mu_eff=0.02, dt=1e-4)], stream=stream)
        ens.set_launch(sweep_grid=sweep_grid, tile_grid=tile_grid)
        with torch.cuda.stream(stream):
            rho, vel, p, _ = I.smooth_primitives(shape, seed=3, amp=0.3, kmax=3)
            Plan(shape, mu_eff=0.02, stream=stream).init_state(rho, vel, p, out=ens.state(0))
            ens.run(1, diag=False, graph=False)
            stream.synchronize()
            t = time.perf_counter()
            ens.run(4, diag=False, graph=False)
            stream.synchronize()
            took.append(time.perf_counter() - t)
        out.append(ens.state(0).clone())
    assert torch.equal(out[0], out[1])
    assert took[1] > 4.0 * took[0], took
