"""The distances that a scene's construction from occupancy hands to its caller
are a copy: the scene never depends on the caller's buffer (shared by builds on
two streams, written again at once), any memory that the copy engine takes will
do, and they are there also where only the scene's part of the call fails.  All
comparisons are of equal bits: one and the same kernel makes every field."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2410_16727_amd import dsopt  # noqa: E402
from workloads import configs, gen, params  # noqa: E402

SHAPE = (61, 70, 83)
VOXEL, ORIGIN = 0.02, (-0.8, -0.7, -0.3)
PROB = configs.problems("A")[0]


def occupancy(seed):
    rng = np.random.default_rng(seed)
    occ = np.zeros(SHAPE, dtype=np.uint8)
    for _ in range(12):
        a = [int(rng.integers(0, n - 8)) for n in SHAPE]
        occ[a[0]:a[0] + 8, a[1]:a[1] + 6, a[2]:a[2] + 7] = 1
    return torch.from_numpy(occ).cuda()


def make_plan():
    return dsopt.Plan(configs.robot("A"), params.DEFAULT, 1, 256 << 20)


def score(pl, scene):
    X = torch.from_numpy(gen.random_trajectories(np.random.default_rng(1), 64, 32, PROB.q_start)).cuda()
    return pl.cost(scene, PROB.q_start, PROB.goal, X).cpu()


def alone(occ):
    """Field and costs of a scene built by itself."""
    pl = make_plan()
    out = torch.zeros(SHAPE, dtype=torch.float32, device="cuda")
    pl.scene_from_occupancy(0, occ, VOXEL, ORIGIN, out=out)
    J = score(pl, 0)
    pl.close()
    return out.cpu(), J


@pytest.mark.parametrize("streams", [1, 2])
def test_scenes_sharing_one_buffer(streams):
    occ = [occupancy(k) for k in (1, 2)]
    want = [alone(o)[1] for o in occ]
    assert bool((want[0] != want[1]).any())
    pl = make_plan()
    out = torch.zeros(SHAPE, dtype=torch.float32, device="cuda")
    st = [torch.cuda.Stream() for _ in range(streams)]
    torch.cuda.synchronize()
    for k in range(2):
        pl.scene_from_occupancy(k, occ[k], VOXEL, ORIGIN, out=out, stream=st[k % streams])
    out.fill_(-1.0)   # on a third stream, ordered with neither build
    torch.cuda.synchronize()
    assert all(bool((score(pl, k) == want[k]).all()) for k in range(2))
    pl.close()


@pytest.mark.parametrize("memory", ["pageable", "pinned", "offset"])
def test_memory_of_the_copy(memory):
    occ = occupancy(3)
    want, J = alone(occ)
    pl = make_plan()
    if memory == "offset":
        buf = torch.zeros(want.numel() + 3, dtype=torch.float32, device="cuda")
        out = buf[1:-2].view(SHAPE)
    else:
        out = torch.zeros(SHAPE, dtype=torch.float32, pin_memory=memory == "pinned")
    pl.scene_from_occupancy(0, occ, VOXEL, ORIGIN, out=out)
    torch.cuda.synchronize()
    assert bool((out.cpu() == want).all())
    if memory == "offset":
        assert float(buf[0]) == 0 and bool((buf[-2:] == 0).all())
    assert bool((score(pl, 0) == J).all())
    pl.close()


@pytest.mark.parametrize("host", [False, True])
def test_distances_without_a_place_for_the_scene(host):
    occ = occupancy(4)
    want, _ = alone(occ)
    pl = make_plan()
    out = torch.zeros(SHAPE, dtype=torch.float32, device="cpu" if host else "cuda")
    with pytest.raises(dsopt.DsError) as e:
        pl.scene_from_occupancy(-1, occ, VOXEL, ORIGIN, out=out)
    assert e.value.code == dsopt.DS_ERR_INVALID
    torch.cuda.synchronize()
    assert bool((out.cpu() == want).all())
    # and the plan's arena is whole: the scene still finds its place
    pl.scene_from_occupancy(0, occ, VOXEL, ORIGIN)
    torch.cuda.synchronize()
    pl.close()


@pytest.mark.parametrize("short", ["plain", "view", "host"])
def test_buffer_without_room_is_refused(short):
    """Before anything is launched: the buffer keeps its values, and the scene
    of that id its own."""
    occ = occupancy(5)
    pl = make_plan()
    pl.scene_from_occupancy(0, occupancy(6), VOXEL, ORIGIN)
    before = score(pl, 0)
    n = occ.numel()
    buf = torch.full((n + 8,), 7.0, dtype=torch.float32, device="cpu" if short == "host" else "cuda")
    out = buf[9:] if short == "view" else buf[:n - 1].clone()
    with pytest.raises(dsopt.DsError) as e:
        pl.scene_from_occupancy(0, occ, VOXEL, ORIGIN, out=out)
    assert e.value.code == dsopt.DS_ERR_INVALID
    torch.cuda.synchronize()
    assert bool((buf == 7.0).all()) and bool((out == 7.0).all())
    assert bool((score(pl, 0) == before).all())
    pl.close()
