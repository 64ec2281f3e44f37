"""Links with different sphere counts, so that the wavefronts and lane groups
of a seed hold different numbers of a link's spheres (none, one, two, several
chunks of four): the optimiser's iterations against the FP64 oracle for every
team size, to the tolerances of the plain lockstep tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2410_16727_amd import dsopt  # noqa: E402
from workloads import configs, gen, params  # noqa: E402

from test_gpu_parity import P, lockstep_check, run_traced  # noqa: E402

COUNTS = {"nine": (9, 9, 9, 9, 8, 8, 8), "mixed": (1, 2, 3, 4, 5, 9, 12)}


class Uneven:
    def __init__(self, counts, waves):
        self.key, self.iters = "B", 12
        self.robot = gen.make_robot(gen.rng_for(0, 0), gen.rng_for(3, 1), COUNTS[counts])
        self.scene = configs.scenes(self.key, only={0})[0]
        self.prob = configs.problems(self.key)[0]
        self.plan = dsopt.Plan(self.robot, dict(P, waves_per_seed=waves), self.iters, 512 << 20)
        self.plan.upload_scene(0, self.scene.grid, self.scene.voxel, self.scene.origin)
        self.O = oracle.Oracle(self.robot, self.scene, params.as_list(), threads=8)


@pytest.mark.parametrize("counts", sorted(COUNTS))
@pytest.mark.parametrize("waves,T", [(1, 13), (1, 40), (2, 13), (2, 30), (2, 40), (4, 13), (4, 30), (4, 40), (8, 40)])
def test_lockstep_uneven_links(counts, waves, T):
    su = Uneven(counts, waves)
    print(f"uneven links {counts} W={waves} T={T}", flush=True)
    seeds, tr = run_traced(su, S=4, T=T, tag=6)
    lockstep_check(su, tr, seeds.shape[0])
    assert np.isfinite(tr["x"]).all()
    su.plan.close()
