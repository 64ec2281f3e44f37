"""The optional terms (self-collision pairs, swept samples) in the optimiser,
for every team size, with the spheres on their links' axes (centres from the
twists alone) and with some off them (centres from the whole frames, shared by
a full team or formed again by the others), lane groups of 16 and 64 lanes,
against the FP64 oracle iteration by iteration, to the tolerances of the plain
lockstep tests."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2410_16727_amd import dsopt  # noqa: E402
from workloads import configs, params  # noqa: E402

from test_gpu_offaxis import offaxis_robot  # noqa: E402
from test_gpu_parity import check_cost_grad, lockstep_check, random_trajs, run_traced  # noqa: E402


class Terms:
    def __init__(self, waves, off, swept):
        self.key = "B"
        self.ps = dict(params.DEFAULT, w_self=50.0, swept_samples=swept, waves_per_seed=waves)
        robot = offaxis_robot(self.key) if off else configs.robot(self.key)
        # larger spheres, so that pairs touch
        self.robot = dataclasses.replace(
            robot, sphere_radius=(robot.sphere_radius * 1.6).astype(np.float32))
        self.scene = configs.scenes(self.key, only={0})[0]
        self.prob = configs.problems(self.key)[0]
        self.iters = 12
        self.plan = dsopt.Plan(self.robot, self.ps, self.iters, 512 << 20)
        self.plan.upload_scene(0, self.scene.grid, self.scene.voxel, self.scene.origin)
        self.O = oracle.Oracle(self.robot, self.scene, params.as_list(self.ps), threads=8)


@pytest.mark.parametrize("waves,off,swept,T", [(1, 0, 1, 13), (2, 0, 1, 13), (4, 0, 1, 50), (8, 0, 1, 13),
                                               (1, 1, 0, 50), (2, 1, 0, 50), (4, 1, 0, 13), (8, 1, 2, 50)])
def test_self_and_swept_lockstep(waves, off, swept, T):
    su = Terms(waves, off, swept)
    print(f"optional terms W={waves} off-axis={off} swept={swept} T={T}", flush=True)
    seeds, tr = run_traced(su, S=4, T=T, tag=5)
    lockstep_check(su, tr, seeds.shape[0])
    res = su.plan.seed_results(5, seeds.shape[0])
    ref = su.O.results(su.prob.q_start, su.prob.goal, tr["x"][-1])
    amb = np.abs(ref["clearance"]) < 1e-5
    for f in ["collision_free", "success", "valid"]:
        assert ((res[f] == ref[f].astype(int)) | amb).all(), f
    assert np.abs(res["clearance"] - ref["clearance"]).max() < 1e-4
    su.plan.close()


@pytest.mark.parametrize("S,T", [(3, 13), (40, 33), (700, 16)])   # teams of 8, 4 and 1
def test_self_offaxis_cost_grad(S, T):
    su = Terms(1, 1, 1)
    check_cost_grad(su, random_trajs(500 + S, S, T, su.prob.q_start))
    su.plan.close()
