"""Plans that gather every sample have kernels of their own for teams of 2 and 4:
whole optimisations bitwise those of the plans that skip, and every sample
counted, with one sphere per copy and link and with several."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import test_gpu_far_skip as far_skip  # noqa: E402


@pytest.mark.parametrize("key,waves", [("A", 2), ("B", 2), ("B", 4), ("D", 2), ("D", 4)])
def test_optimisation_identical(key, waves):
    far_skip.test_optimisation_identical_and_gathers_counted(key, waves)
