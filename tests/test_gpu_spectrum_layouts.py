"""The spectrum's transforms and intermediate layouts at the sizes where they change: every
radix chain of the register path (8 to 1024), partial runs of kx, line gaps, the wide blocks
of large boxes, odd and prime lengths along each direction, and shell counts that leave fewer
histograms than waves.

Tolerance: an FFT's relative error in the 2-norm is at most about 5 eps log2(n3) (3e-14 here),
so shells and moments agree to 1e-12 of the total energy.
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2211_16718_amd.api import Plan  # noqa: E402


@pytest.mark.parametrize("shape,length", [  # (nz, ny, nx)
    ((16, 8, 64), None),
    ((1024, 16, 8), None),
    ((8, 1024, 32), None),
    ((128, 128, 8), None),                   # line gaps, 256 threads
    ((256, 128, 128), None),                 # 512 threads
    ((64, 64, 1024), None),
    ((129, 131, 9), None),                   # line gaps, generic radices, odd nx
    ((11, 503, 10), None),
    ((2047, 8, 8), None),
    ((2047, 8, 8), (2.0, 2.0, 1.6075)),      # the most shells: one histogram
    ((1024, 8, 8), (2.0, 2.0, 1.25)),        # 2600 shells
])
def test_spectrum_layouts(shape, length):
    from oracle import spectrum as S

    print(f"[case] spectrum layout {shape} L={length}", flush=True)
    length = length or (2 * math.pi,) * 3
    rng = np.random.default_rng(sum(shape))
    rho = 1.0 + 0.2 * rng.random(shape)
    vel = rng.normal(size=(3,) + shape)
    plan = Plan(shape, length=length)
    u = plan.init_state(rho, vel, np.full(shape, 2.0))
    E, mom = plan.spectrum(u)
    Er, tot, m2 = S.spectrum(u.cpu().numpy(), length)
    assert E.shape == Er.shape
    np.testing.assert_allclose(E.cpu().numpy(), Er, rtol=0, atol=1e-12 * tot)
    assert mom[0].item() == pytest.approx(tot, rel=1e-12)
    assert mom[1].item() == pytest.approx(m2, rel=1e-12)
