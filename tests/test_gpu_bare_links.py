"""Optimiser iterations of robots with links that carry no sphere -- one, three
or six of the seven, the first or the last among them -- for every team size and
lane group, against the FP64 oracle iteration by iteration, to the tolerances of
the plain lockstep tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import test_gpu_uneven_links as uneven  # noqa: E402
from test_gpu_parity import lockstep_check, run_traced  # noqa: E402

COUNTS = {"one": (4, 4, 0, 9, 4, 4, 4), "three": (0, 1, 17, 3, 0, 9, 0), "six": (0, 0, 0, 0, 0, 20, 0)}


@pytest.mark.parametrize("counts", sorted(COUNTS))
@pytest.mark.parametrize("waves,T", [(1, 13), (1, 30), (1, 50), (2, 13), (2, 50), (4, 13), (4, 30), (8, 13), (8, 50)])
def test_lockstep_bare_links(monkeypatch, counts, waves, T):
    monkeypatch.setitem(uneven.COUNTS, counts, COUNTS[counts])
    su = uneven.Uneven(counts, waves)
    print(f"bare links {counts} W={waves} T={T}", flush=True)
    seeds, tr = run_traced(su, S=5, T=T, tag=6)
    lockstep_check(su, tr, seeds.shape[0])
    assert np.isfinite(tr["x"]).all()
    su.plan.close()
