"""Weight gradient of the second convolution, whose deltas enter a sparse matrix instruction as pooled values with their places: against
the oracle where rows and columns of windows don't fill its steps (images narrower than 16 pixels, of one and of several steps a row,
tiles of rows with a shorter last one), channels beyond a block, waves that share a block and waves that don't, both filter sizes."""
import pytest

from test_gpu_grad_cnn import B  # noqa: F401  (the fixture)
from test_gpu_second_conv import test_second_layer_matches_oracle as second_layer

pytestmark = pytest.mark.gpu

# input channels, height, width, channels 1 and 2, filter, dense, classes; batch
SHAPES = [((1, 8, 8, 4, 33, 3, 6, 5), 9), ((1, 8, 8, 5, 6, 5, 6, 5), 70), ((2, 12, 72, 5, 7, 3, 6, 5), 3), ((1, 96, 12, 3, 5, 5, 6, 5), 3),
          ((1, 64, 64, 4, 6, 5, 6, 5), 2), ((3, 28, 36, 9, 34, 5, 6, 5), 2), ((1, 20, 20, 33, 64, 3, 6, 5), 4), ((1, 44, 28, 12, 20, 3, 6, 5), 3)]


@pytest.mark.parametrize("shape,batch", SHAPES, ids=["-".join(map(str, s[0])) + f"-b{s[1]}" for s in SHAPES])
def test_weight_gradient_of_pooled_deltas(B, orc, shape, batch):  # noqa: F811
    second_layer(B, orc, shape, batch)
