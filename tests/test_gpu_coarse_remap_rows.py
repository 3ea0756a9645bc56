"""GPU: the remapping by rows of large grids with a far field (rows of 59, 60 and 257
cells; rows that would leave lanes idle take the other form at 41 and 100)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import test_gpu_coarse_remap as remap  # noqa: E402


@pytest.mark.parametrize("shape,B", [((230, 390, 59), 4), ((301, 300, 60), 5), ((143, 143, 257), 3),
                                     ((220, 240, 100), 6)])
def test_far_field(shape, B):
    remap.test_means_of_the_blocks(shape, B, True)
