"""Cost and gradient against the FP64 oracle where the sampling of a link's
spheres can go wrong: links without spheres, with one, with more than a chunk
holds and unevenly many, on and off the link's axis, for every team size the
cost calls choose (8, 4, 2 and 1 wavefronts per seed, by the number of seeds)
and every lane group; and joint angles on both sides of 2^17, where the
kinematics changes from the short argument reduction to the long one.
Tolerances are those of test_gpu_parity."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2410_16727_amd import dsopt  # noqa: E402
from workloads import configs, gen, params  # noqa: E402

from test_gpu_parity import COST_RTOL, GRAD_RTOL, grad_check, say  # noqa: E402

TABLES = {
    "uneven": (0, 1, 17, 3, 0, 9, 0),
    "last": (0, 0, 0, 0, 0, 0, 1),
    "nine": (9, 9, 9, 9, 8, 8, 8),
    "many": (18, 18, 18, 18, 18, 18, 20),
}


def arm(table, off_axis):
    r = gen.make_robot(gen.rng_for(*configs.ARM_STREAM), gen.rng_for(9, 1), table)
    if off_axis:
        off = r.sphere_offset.copy()
        off[r.sphere_link % 2 == 1, 0] = 0.02
        r = dataclasses.replace(r, sphere_offset=off)
    return r


@pytest.mark.parametrize("S", [3, 600, 1100, 2100])
@pytest.mark.parametrize("T", [16, 23, 50])
@pytest.mark.parametrize("table,off_axis", [("uneven", False), ("uneven", True), ("last", False),
                                            ("nine", False), ("nine", True), ("many", True)])
def test_cost_grad(table, off_axis, T, S):
    robot = arm(TABLES[table], off_axis)
    prob = configs.problems("D")[0]
    scene = configs.scenes("D", only={prob.scene})[prob.scene]
    plan = dsopt.Plan(robot, params.DEFAULT, 1, 256 << 20)
    plan.upload_scene(0, scene.grid, scene.voxel, scene.origin)
    O = oracle.Oracle(robot, scene, params.as_list(), threads=8)
    say(f"sphere table {table} off-axis {off_axis} T={T} S={S}")
    X = gen.random_trajectories(np.random.default_rng(T), 3, T, prob.q_start, scale=0.5)
    many = torch.from_numpy(np.resize(X, (S, T, 7))).cuda()
    J, G = plan.cost_grad(0, prob.q_start, prob.goal, many)
    J2 = plan.cost(0, prob.q_start, prob.goal, many).cpu().numpy()
    J, G = J.cpu().numpy(), G.cpu().numpy()
    plan.close()
    ref = O.cost(prob.q_start, prob.goal, X.astype(np.float64), grad=True, absg=True)
    for s in range(min(S, 3)):
        # every repetition of a trajectory has the first one's bits
        assert np.all(J[s::3] == J[s]) and np.all(G[s::3] == G[s]) and np.all(J2[s::3] == J2[s])
        assert abs(J[s] - ref["J"][s]) <= COST_RTOL * ref["J"][s]
        assert abs(J2[s] - ref["J"][s]) <= COST_RTOL * ref["J"][s]
        worst, need = grad_check(O, prob, X[s], G[s], ref["G"][s], ref["A"][s])
        assert worst <= GRAD_RTOL, (s, worst, need)


@pytest.mark.parametrize("S", [3, 2100])
def test_angles_around_the_long_reduction(S):
    """Angles at, below and far above 2^17 in some lanes of some seeds, the
    others ordinary; the limit penalty is off (it would drown the rest)."""
    robot = configs.robot("A")
    prob = configs.problems("A")[0]
    scene = configs.scenes("A", only={0})[0]
    p = dict(params.DEFAULT, w_limit=0.0, lambda_v=0.0, lambda_a=0.0, lambda_j=0.0)
    plan = dsopt.Plan(robot, p, 1, 64 << 20)
    plan.upload_scene(0, scene.grid, scene.voxel, scene.origin)
    O = oracle.Oracle(robot, scene, params.as_list({k: p[k] for k in ("w_limit", "lambda_v", "lambda_a",
                                                                      "lambda_j")}), threads=8)
    X = gen.random_trajectories(np.random.default_rng(5), 3, 32, prob.q_start, scale=0.5)
    two17 = np.float32(2 ** 17)
    X[1, 7, :3] = (two17, np.nextafter(two17, np.float32(0)), -two17)
    X[2, 31, 6] = 3.0e6
    many = torch.from_numpy(np.resize(X, (S, 32, 7))).cuda()
    J = plan.cost(0, prob.q_start, prob.goal, many).cpu().numpy()
    plan.close()
    ref = O.cost(prob.q_start, prob.goal, X.astype(np.float64))["J"]
    for s in range(3):
        assert np.all(J[s::3] == J[s])
        assert abs(J[s] - ref[s]) <= COST_RTOL * ref[s]
