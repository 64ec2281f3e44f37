"""The optional terms (self-collision pairs, swept samples) in the cost,
gradient and guidance calls for every team size that these choose by the number
of seeds (3: eight wavefronts per seed, 600: four, 1100: two, 2101: one, with a
last workgroup that has a single seed), against the FP64 oracle.  A few
trajectories fill the batch in turn: every repetition has the first one's bits.
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

from test_gpu_offaxis import offaxis_robot  # noqa: E402
from test_gpu_parity import (AMB_TOL, COST_RTOL, GRAD_C, GRAD_RTOL, KC, KETA, U32,  # noqa: E402
                             grad_check, say)

N = 3   # distinct trajectories


class Terms:
    def __init__(self, off_axis, w_self, swept):
        ps = dict(params.DEFAULT, w_self=w_self, swept_samples=swept)
        robot = offaxis_robot("B") if off_axis else configs.robot("B")
        # larger spheres, so that pairs touch
        self.robot = dataclasses.replace(robot, sphere_radius=(robot.sphere_radius * 1.6).astype(np.float32))
        scene = configs.scenes("B", only={0})[0]
        self.prob = configs.problems("B")[0]
        self.plan = dsopt.Plan(self.robot, ps, 1, 512 << 20)
        self.plan.upload_scene(0, scene.grid, scene.voxel, scene.origin)
        self.O = oracle.Oracle(self.robot, scene, params.as_list(ps), threads=8)

    def trajectories(self, S, T):
        X = gen.random_trajectories(np.random.default_rng(70 + T), N, T, self.prob.q_start)
        return X, np.resize(X, (S, T, 7))


def repeats(a):
    """Every repetition of a trajectory has the first one's bits."""
    return all(np.all(a[s::N] == a[s]) for s in range(N))


@pytest.mark.parametrize("S", [3, 600, 1100, 2101])
@pytest.mark.parametrize("T", [13, 32, 47])
@pytest.mark.parametrize("off_axis,w_self,swept", [(False, 50.0, 2), (True, 50.0, 1), (False, 50.0, 0), (True, 0.0, 2),
                                                  (False, 0.0, 8)])
def test_cost_grad(off_axis, w_self, swept, T, S):
    say(f"optional terms off-axis={off_axis} w_self={w_self} swept={swept} T={T} S={S}")
    su = Terms(off_axis, w_self, swept)
    X, many = su.trajectories(S, T)
    many = torch.from_numpy(many).cuda()
    J, G = su.plan.cost_grad(0, su.prob.q_start, su.prob.goal, many)
    J2 = su.plan.cost(0, su.prob.q_start, su.prob.goal, many).cpu().numpy()
    J, G = J.cpu().numpy(), G.cpu().numpy()
    su.plan.close()
    assert repeats(J) and repeats(G) and repeats(J2)
    ref = su.O.cost(su.prob.q_start, su.prob.goal, X.astype(np.float64), grad=True, absg=True)
    for s in range(N):
        assert abs(J[s] - ref["J"][s]) <= COST_RTOL * ref["J"][s]
        assert abs(J2[s] - ref["J"][s]) <= COST_RTOL * ref["J"][s]
        worst, need = grad_check(su.O, su.prob, X[s], G[s], ref["G"][s], ref["A"][s])
        assert worst <= GRAD_RTOL, (s, worst, need)


@pytest.mark.parametrize("S", [3, 600, 1100, 2101])
@pytest.mark.parametrize("off_axis,w_self,swept,T", [(False, 50.0, 2, 32), (True, 50.0, 1, 47), (False, 50.0, 0, 13)])
def test_guide(off_axis, w_self, swept, T, S):
    """Two steps in one call have the bits of two calls, and each step is the
    oracle's from the same trajectories."""
    say(f"guidance with optional terms off-axis={off_axis} w_self={w_self} swept={swept} T={T} S={S}")
    alpha = 2e-5
    su = Terms(off_axis, w_self, swept)
    _, many = su.trajectories(S, T)
    two = torch.from_numpy(many).cuda()
    J = su.plan.guide(0, su.prob.q_start, su.prob.goal, two, alpha, 2).cpu().numpy()
    at = torch.from_numpy(many).cuda()
    for k in range(2):
        X = at[:N].cpu().numpy().astype(np.float64)
        su.plan.guide(0, su.prob.q_start, su.prob.goal, at, alpha, 1)
        got = at.cpu().numpy()
        assert repeats(got)
        ref = su.O.cost(su.prob.q_start, su.prob.goal, X, grad=True, absg=True)
        for s in range(N):
            amb, _ = su.O.ambiguity(X[s], AMB_TOL)
            fb, _ = su.O.fp32_bound(su.prob.q_start, su.prob.goal, X[s], KC, KETA)
            tol = alpha * (GRAD_RTOL * np.abs(ref["G"][s]).max() + GRAD_C * U32 * ref["A"][s] + amb + fb) + \
                2 * U32 * np.abs(X[s])
            assert (np.abs(got[s] - (X[s] - alpha * ref["G"][s])) <= tol).all(), (k, s)
    su.plan.close()
    assert np.array_equal(two.cpu().numpy(), got) and repeats(J)
    ref = su.O.cost(su.prob.q_start, su.prob.goal, got[:N].astype(np.float64))["J"]
    assert (np.abs(J[:N] - ref) <= COST_RTOL * ref).all()
