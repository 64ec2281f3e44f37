"""Records and coarse table of grids whose rows of blocks are cut into parts
(rows of even and odd length, blocks of 4, 8 and 16 cells), whole where one per
workgroup fills the CUs evenly, or joined, by rows and by layers: every record and every level against numpy, exactly."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import test_gpu_scene_build as build  # noqa: E402


@pytest.mark.parametrize("dims", [
    (2, 2, 700), (3, 5, 90), (5, 4, 66), (9, 6, 139),                      # layers joined
    (2, 300, 7), (5, 70, 41), (12, 90, 10), (61, 23, 9), (129, 30, 6),     # rows joined
    (130, 7, 6), (134, 70, 5), (300, 130, 120), (290, 131, 121),           # parts, 4 and 8 cells
    (1470, 1460, 2), (1450, 1470, 2),                                      # parts, 16 cells
    (148, 145, 111), (158, 145, 111),                                      # whole rows, odd and even
    (140000, 3, 3), (20006, 4, 60), (2300, 3, 520), (9000, 10, 70)])       # parts of thin rows
def test_records_and_table(dims):
    print(f"grid {dims}", flush=True)
    build.test_records_and_table(dims)
