"""The fused head on 17 to 32 classes, two tiles of the matrix instruction: gradients against the oracle (one chunk of samples and several,
several workgroups to a chunk, forward products in parts, 33 classes on the kernels beyond it), and rounds that average on the way against
a gradient pass and an averaging pass, bit for bit."""
import pytest

from test_gpu_average import test_average_on_the_way_is_the_average as average_on_the_way
from test_gpu_grad_mlp import B, check_gradients  # noqa: F401  (B: the fixture)

pytestmark = pytest.mark.gpu

GRADIENTS = [([784, 17], 32, 2, "xent"), ([301, 32], 5, 2, "mse"), ([20, 260, 31], 70, 3, "xent"), ([20, 516, 31], 64, 3, "mse"), ([33, 29, 30], 17, 3, "mse"), ([64, 48, 25], 300, 3, "xent"),
             ([1605, 36, 20], 30, 3, "mse"), ([40, 24, 33], 40, 3, "xent")]
AVERAGE = [([784, 26], 32, "xent", 8, 64), ([101, 17], 64, "mse", 9, 1), ([256, 32], 600, "xent", 6, 64), ([300, 92, 20], 32, "mse", 17, 64)]


@pytest.mark.parametrize("dims,batch,n,loss", GRADIENTS, ids=["-".join(map(str, s[0])) + f"-b{s[1]}" for s in GRADIENTS])
def test_gradients_match_oracle(B, orc, dims, batch, n, loss):  # noqa: F811
    check_gradients(B, orc, dims, batch, n, loss, expect={"fc_head_kernel" if dims[-1] <= 32 else "softmax_loss_kernel"})


@pytest.mark.parametrize("dims,batch,loss,n,pad", AVERAGE, ids=["-".join(map(str, s[0])) + f"-b{s[1]}" for s in AVERAGE])
def test_average_on_the_way(B, dims, batch, loss, n, pad):  # noqa: F811
    average_on_the_way(B, dims, batch, loss, n, pad, "each")


@pytest.mark.parametrize("dims,batch,n,head", [([978, 17], 64, 32, True), ([978, 17], 64, 33, False), ([784, 20], 48, 42, True), ([784, 20], 48, 43, False),
                                               ([256, 20], 64, 64, True), ([40, 600, 20], 33, 64, True)])
def test_chunks_of_a_short_batch(B, orc, dims, batch, n, head):  # noqa: F811
    """A short batch that does not fit the head's LDS whole, in chunks of one workgroup to a compute unit, on half of the chip and beyond."""
    check_gradients(B, orc, dims, batch, n, "xent", expect={"fc_head_kernel" if head else "softmax_loss_kernel"})
