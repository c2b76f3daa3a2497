"""psi bricks with rows of 32 cells on further sides: the smallest one that takes bricks (80: a
row that overhangs by half in z, and none in y) and 112 (overhang in z alone), next to the
side of 88 (overhang in y and z).  Same bounds as the other sides' tests."""
import pytest

from paper_2501_13046_amd import grtmg as g
from test_gpu_bricks import RULES
from test_gpu_bricks import test_pass_and_defect as pass_and_defect
from test_gpu_bricks import test_residual_without_w as residual_without_w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,levels", [(80, 5), (112, 5)])
@pytest.mark.parametrize("bc", RULES)
def test_rows_of_32(n, levels, bc):
    for precision in (g.PREC_FP32_IR, g.PREC_FP64):
        pass_and_defect(n, levels, bc, precision)
    residual_without_w(n, levels, bc)
