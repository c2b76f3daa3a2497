"""Large convolutions whose bricks the eight XCDs' blocks walk in uneven shares, against the
FP64 oracle: more bricks than blocks, a number of bricks that 8 does not divide, and several
channel tiles.  Same bounds as the smaller sides' tests."""
import pytest

from test_gpu_nn_bricks import test_convolution_on_any_side as convolution

pytestmark = pytest.mark.gpu


# 18 x 9 x 9 bricks, 1458 of one tile for 1024 blocks; with slices of 32 channels 14 x 7 x 7 = 686,
# two tiles, 256 blocks each, and 13 x 7 x 7 = 637, four tiles, 128 blocks each
@pytest.mark.parametrize("n,cin,cout", [(72, 8, 4), (56, 32, 20), (52, 32, 52)])
def test_uneven_shares(n, cin, cout):
    convolution(n, cin, cout, False)
