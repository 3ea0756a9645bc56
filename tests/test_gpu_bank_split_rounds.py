"""GPU: the bank apply in parts near the tile counts at which it is left whole: 160
to 320 tiles against the apply in one part (a budget without room for the parts).  Bar as in the other test of the parts: W^3 2^-53 relative."""
import pytest

import test_gpu_bank_split as split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,r,prec,esz", [
    ((33, 40, 70), 8, split.fd.FP16_BANK, 2), ((33, 50, 70), 8, split.fd.FP16_BANK, 2),
    ((17, 80, 66), 3, split.fd.FP32, 4), ((9, 64, 70), 2, split.fd.FP64, 8), ((33, 65, 65), 4, split.fd.BF16_BANK, 2),
    ((31, 80, 64), 5, split.fd.FP64, 8)])
def test_parts_equal_whole(shape, r, prec, esz):
    split.test_parts_equal_whole(shape, r, prec, esz)
