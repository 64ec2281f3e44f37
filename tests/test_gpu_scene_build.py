"""Scene construction at the sizes where its tiling can go wrong: the
distance transform against the oracle's brute-force definition (tiles of 32
lines, gaps of 4, 16 and 64 voxels, row masks of 64), and the resident form
-- cell records and coarse table -- against the same written with numpy
(rows of 32 blocks, bytes shared by two rows).  Squared distances are whole
numbers on both sides, so only the root and the scaling round (two
operations, 2^-23 each at most); records and levels are exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2410_16727_amd import dsopt  # noqa: E402
from workloads import configs, params  # noqa: E402


def occupancy(shape, kind, rng):
    occ = np.zeros(shape, dtype=np.uint8)
    if kind == "sparse":
        occ[tuple(rng.integers(0, n, 3) for n in shape)] = 1
    elif kind == "dense":
        occ[:] = 1
        occ[tuple(rng.integers(0, n, 3) for n in shape)] = 0
    elif kind == "boxes":
        for _ in range(4):
            a = [int(rng.integers(0, n)) for n in shape]
            b = [min(n, o + int(rng.integers(1, 2 + n // 3))) for o, n in zip(a, shape)]
            occ[a[0]:b[0], a[1]:b[1], a[2]:b[2]] = 3   # any nonzero byte is occupied
        occ.reshape(-1)[0] = 0
    else:
        occ[rng.random(shape) < 0.3] = 1
        occ.reshape(-1)[:2] = (1, 0)
    return occ


@pytest.mark.parametrize("kind", ["sparse", "dense", "boxes", "noise"])
@pytest.mark.parametrize("shape", [(2, 2, 2), (5, 16, 65), (17, 63, 32), (64, 65, 33), (31, 4, 128),
                                   (130, 3, 5), (3, 257, 2), (2, 3, 1024), (2, 1024, 3),
                                   (1024, 2, 3)])
def test_distance_transform(shape, kind):
    rng = np.random.default_rng(sum(shape) + len(kind))
    occ = occupancy(shape, kind, rng)
    pl = dsopt.Plan(configs.robot("A"), params.DEFAULT, 1, 256 << 20)
    out = torch.zeros(shape, dtype=torch.float32, device="cuda")
    pl.scene_from_occupancy(0, torch.from_numpy(occ).cuda(), 0.01, (0.0, 0.0, 0.0), out=out)
    torch.cuda.synchronize()
    pl.close()
    d = out.cpu().numpy().astype(np.float64).reshape(-1)
    idx = rng.choice(occ.size, min(occ.size, 3000), replace=False)
    ref = oracle.esdf_from_occupancy(occ, np.float32(0.01), which=idx, threads=8)
    assert np.all(np.abs(d[idx] - ref) <= 2.0 ** -22 * np.abs(ref))
    assert np.array_equal(d < 0, occ.reshape(-1) != 0)


@pytest.mark.parametrize("occupied", [False, True])
def test_field_without_the_other_kind(occupied):
    """A grid with no occupied (no free) voxel: distances of at least 1e9
    voxels, of the right sign."""
    occ = torch.full((9, 40, 70), 1 if occupied else 0, dtype=torch.uint8, device="cuda")
    pl = dsopt.Plan(configs.robot("A"), params.DEFAULT, 1, 256 << 20)
    out = torch.zeros(occ.shape, dtype=torch.float32, device="cuda")
    pl.scene_from_occupancy(0, occ, 0.5, (0.0, 0.0, 0.0), out=out)
    torch.cuda.synchronize()
    pl.close()
    assert bool((out * (-1 if occupied else 1) >= 0.5e9).all())


def levels(v, cq, shift, blocks):
    """[cdz, cdy, cdx] levels of the node values v [nz, ny, nx]."""
    out = np.zeros(blocks, dtype=np.uint8)
    b = 1 << shift
    for k, j, i in np.ndindex(*blocks):
        m = np.nanmin(np.append(v[k * b:(k + 1) * b + 1, j * b:(j + 1) * b + 1,
                                  i * b:(i + 1) * b + 1], np.finfo(np.float32).max))
        if m >= 0:
            out[k, j, i] = max(L for L in range(16) if np.float32(L) * cq <= m)
    return out


@pytest.mark.parametrize("dims", [(2, 2, 2), (6, 5, 4), (64, 33, 30), (37, 21, 13), (130, 9, 8),
                                  (133, 6, 10), (400, 4, 3), (6, 130, 131), (145, 137, 131)])
def test_records_and_table(dims):
    """Every record and every table entry of a scene, read from the arena
    (the table follows the records, at the next multiple of 256 bytes)."""
    nx, ny, nz = dims
    rng = np.random.default_rng(nx)
    v = rng.uniform(-0.02, 0.3, (nz, ny, nx)).astype(np.float32)
    v += rng.uniform(0, 0.2, ((nz + 3) // 4, (ny + 3) // 4, (nx + 3) // 4)).astype(np.float32).repeat(
        4, 0).repeat(4, 1).repeat(4, 2)[:nz, :ny, :nx]
    v[0, 0, 0] = np.nan
    robot = configs.robot("A")
    pl = dsopt.Plan(robot, params.DEFAULT, 1, 256 << 20)
    pl.upload_scene(0, v, 0.02, (0.0, 0.0, 0.0))
    torch.cuda.synchronize()
    rec = np.stack([v[dz:nz - 1 + dz, dy:ny - 1 + dy, dx:nx - 1 + dx]
                    for dz in (0, 1) for dy in (0, 1) for dx in (0, 1)], -1)
    want = np.ascontiguousarray(rec).reshape(-1).view(np.uint8)
    raw = pl.arena[:(1 << 16) + want.size + (1 << 15)].cpu().numpy()
    pl.close()
    # the records come before the staged copy of the values
    at = [o for o in range(0, 1 << 16, 256) if np.array_equal(raw[o:o + 32], want[:32])]
    assert at
    assert np.array_equal(raw[at[0]:at[0] + want.size], want)
    shift = 2
    while np.prod([-(-(n - 1) // (1 << shift)) for n in dims]) > 32768:
        shift += 1
    blocks = [-(-(n - 1) // (1 << shift)) for n in (nz, ny, nx)]
    cq = (robot.sphere_radius.max() + (np.float32(0.02) + np.float32(1e-5))) / np.float32(8)
    want = levels(v, cq, shift, blocks).reshape(-1)
    table = raw[at[0] + -(-rec.size * 4 // 256) * 256:]
    got = np.stack([table & 15, table >> 4], 1).reshape(-1)[:want.size]
    assert np.array_equal(got, want)
