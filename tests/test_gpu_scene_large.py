"""Records and coarse table of grids whose records exceed 256 MB, where they are
made by a kernel each or in one pass (by how well the one pass fills its lanes):
rows of blocks that are one tile, joined rows, parts of even and odd rows, blocks
of 8 and 16 cells.  Every record against torch and every level against numpy,
exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2410_16727_amd import dsopt  # noqa: E402
from workloads import configs, params  # noqa: E402

from test_gpu_scene_build import levels  # noqa: E402


@pytest.mark.parametrize("dims", [
    (204, 203, 207), (66, 517, 260), (22, 826, 489), (1424, 10, 700), (40, 600, 380),   # a kernel each, 8 cells
    (40, 600, 700), (700, 600, 40), (3, 3000, 1500), (11, 1203, 1010), (74, 979, 257),  # ... and 16
    (256, 256, 256), (385, 150, 156), (401, 401, 61)])                                  # in one pass
def test_records_and_table(dims):
    nx, ny, nz = dims
    print(f"grid {dims}", flush=True)
    rng = np.random.default_rng(nx)
    v = rng.uniform(-0.02, 0.3, (nz, ny, nx)).astype(np.float32)
    v += rng.uniform(0, 0.2, (nz // 16 + 1, ny // 16 + 1, nx // 16 + 1)).astype(np.float32).repeat(
        16, 0).repeat(16, 1).repeat(16, 2)[:nz, :ny, :nx]
    v[0, 0, 0] = np.nan
    robot = configs.robot("A")
    n = (nx - 1) * (ny - 1) * (nz - 1) * 32
    assert n > 256 << 20
    pl = dsopt.Plan(robot, params.DEFAULT, 1, n + (64 << 20))
    V = torch.from_numpy(v).cuda()
    pl.upload_scene(0, V, 0.02, (0.0, 0.0, 0.0))
    torch.cuda.synchronize()
    want = torch.stack([V[dz:nz - 1 + dz, dy:ny - 1 + dy, dx:nx - 1 + dx]
                        for dz in (0, 1) for dy in (0, 1) for dx in (0, 1)], -1).view(-1).view(torch.uint8)
    head = [o for o in range(0, 1 << 16, 256) if torch.equal(pl.arena[o:o + 32], want[:32])]
    assert head and torch.equal(pl.arena[head[0]:head[0] + n], want)
    shift = 2
    while np.prod([-(-(d - 1) // (1 << shift)) for d in dims]) > 32768:
        shift += 1
    blocks = [-(-(d - 1) // (1 << shift)) for d in (nz, ny, nx)]
    at = head[0] + -(-n // 256) * 256
    table = pl.arena[at:at + (1 << 14)].cpu().numpy()
    pl.close()
    cq = (robot.sphere_radius.max() + (np.float32(0.02) + np.float32(1e-5))) / np.float32(8)
    want = levels(v, cq, shift, blocks).reshape(-1)
    got = np.stack([table & 15, table >> 4], 1).reshape(-1)[:want.size]
    assert np.array_equal(got, want)
