"""The two ends of a perceptron's gradient, against the oracle: the loss of more than sixteen classes (sixteen lanes to a sample: class counts on
both sides of their multiples, up to 32 in the fused head and from 33 on in a kernel of its own, batches of one sample, of one workgroup and of several), and the fused head on few workers with wide inputs, where
several workgroups share a chunk of samples (column runs of 256, ragged ends, one layer and two, one chunk and several)."""
import pytest

from test_gpu_grad_mlp import B, check_gradients  # noqa: F401  (B: the fixture)

pytestmark = pytest.mark.gpu

LOSS = [([12, 17], 1, 3, "xent"), ([12, 32], 64, 2, "mse"), ([9, 33], 257, 2, "xent"), ([20, 11, 100], 65, 3, "mse"), ([5, 31], 600, 2, "mse"),
        ([12, 33], 1, 3, "xent"), ([12, 48], 64, 2, "mse"), ([5, 47], 600, 2, "mse"), ([5, 63], 130, 2, "xent")]
HEAD = [([784, 10], 32, 2, "xent"), ([301, 7], 5, 2, "mse"), ([1027, 16], 33, 1, "xent"), ([513, 1], 64, 3, "xent"), ([20, 516, 10], 70, 2, "xent"),
        ([258, 9], 200, 2, "mse"), ([300, 5], 17, 9, "xent"), ([784, 10], 64, 7, "mse")]


@pytest.mark.parametrize("dims,batch,n,loss", LOSS + HEAD, ids=lambda v: "-".join(map(str, v)) if isinstance(v, list) else str(v))
def test_gradients_match_oracle(B, orc, dims, batch, n, loss):  # noqa: F811
    check_gradients(B, orc, dims, batch, n, loss)
