"""The autotuner on a batch small enough to run its stages side by side: the launched grids,
which those launches do not have, are neither timed nor taken from an older cache, and a
cache entry is that of the batch's kind (viscous or not, boxes of the size)."""
import json

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2211_16718_amd.api import Ensemble  # noqa: E402


def tuned(path, nbox, mu):
    ens = Ensemble([dict(shape=(16, 16, 16), mu_eff=mu, dt=1e-4) for _ in range(nbox)])
    ens.u.view(-1).copy_(torch.rand(ens.u.numel(), device=ens.u.device, dtype=ens.dtype) + 1.0)
    ens.autotune(str(path))
    assert [ens.get_launch(i)[1:] for i in range(nbox)] == [(0, 0)] * nbox
    return json.loads(path.read_text())


def test_small_batches_are_tuned_by_kind_and_without_grids(tmp_path):
    print("[case] autotune of small batches", flush=True)
    path = tmp_path / "tiles.json"
    first = tuned(path, 2, 0.02)
    seg = [k for k in first if k.endswith("|seg")]
    assert len(seg) == 1
    # grids that an older tuner left behind are not used
    assert [v for k, v in first.items() if "|grid|" in k] == [0]
    path.write_text(json.dumps({k: (11 if "|grid|" in k else v) for k, v in first.items()}, indent=2))
    assert tuned(path, 2, 0.02) == first
    # other kinds get entries of their own
    assert len([k for k in tuned(path, 3, 0.02) if k.endswith("|seg")]) == 2
    assert len([k for k in tuned(path, 2, 0.0) if k.endswith("|seg")]) == 3
