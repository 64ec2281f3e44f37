"""The distance transform on both sides of the line between its narrow
workgroups (8 lines, where those of 32 would be 64 or fewer and the lines are
longer than 32) and the others, in the pass along x and y and in that along z: short and long lines, rows that end
inside a tile of 8 or a word of 32, against the oracle's brute-force definition
to the rounding of the root and the scaling."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import test_gpu_scene_build as build  # noqa: E402


@pytest.mark.parametrize("kind", ["sparse", "boxes", "noise"])
@pytest.mark.parametrize("shape", [
    (64, 3, 31), (65, 3, 31), (32, 130, 40), (33, 130, 40),     # 64 and 65, 64 and 66 tiles in x and y
    (30, 32, 50), (30, 33, 50),                                 # lines of 32 and 33
    (2, 1024, 1001), (2, 1021, 1024), (3, 600, 705),            # long lines along y: narrow, narrow, not
    (70, 64, 32), (70, 33, 63), (1024, 61, 33), (1023, 64, 33)])  # along z: 64, 65, 63 and 66 groups of lines
def test_distance_transform(shape, kind):
    print(f"grid {shape} {kind}", flush=True)
    build.test_distance_transform(shape, kind)
