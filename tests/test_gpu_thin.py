"""Gradients of fully connected layers on short batches of any width against the oracle: reductions and outputs on both sides of the
steps of 16 and of a lane's four, batches on both sides of the blocks of 64 samples and of the steps of 36 and 32, outputs narrower than a
lane's pair, forward products in parts that the head adds."""
import pytest

from test_gpu_grad_mlp import B, check_gradients  # noqa: F401  (B: the fixture)

pytestmark = pytest.mark.gpu

# dims, batch, workers, kernels that have to run
SHAPES = [([4, 2, 3], 1, 3, {"mlp_thin_forward", "mlp_wgrad_kernel"}), ([5, 5, 4], 3, 3, {"mlp_thin_forward", "mlp_wgrad_kernel"}),
          ([15, 31, 5], 16, 3, {"mlp_thin_forward", "mlp_wgrad_kernel"}), ([17, 33, 6], 17, 3, {"mlp_thin_forward", "mlp_wgrad_kernel"}),
          ([130, 65, 63, 7], 65, 3, {"mlp_thin_forward", "mlp_thin_dgrad", "mlp_wgrad_kernel"}),
          ([47, 34, 35, 29, 20], 104, 3, {"mlp_thin_forward", "mlp_thin_dgrad", "mlp_wgrad_kernel"}),
          ([47, 37, 18, 10], 105, 3, {"mlp_thin_forward", "mlp_thin_dgrad", "mlp_wgrad_kernel"}), ([37, 26, 10], 108, 3, {"mlp_thin_forward", "mlp_wgrad_kernel"}),
          ([47, 37, 18, 10], 109, 3, {"mlp_thin_forward", "mlp_thin_dgrad", "mlp_wgrad_kernel"}),
          ([21, 6, 5, 10], 255, 4, {"mlp_thin_forward", "mlp_thin_dgrad", "mlp_wgrad_kernel"}),
          ([1605, 36, 10], 30, 3, {"mlp_thin_forward", "mlp_wgrad_kernel"}), ([2063, 40, 10], 80, 3, {"mlp_thin_forward", "mlp_wgrad_kernel"}),
          ([333, 77, 55, 17], 60, 12, {"mlp_thin_forward", "mlp_thin_dgrad", "mlp_wgrad_kernel"}),
          ([3, 9, 4], 20, 3, set()), ([9, 1, 4], 20, 3, set())]           # too narrow: the GEMM kernels


@pytest.mark.parametrize("dims,batch,n,kernels", SHAPES, ids=["-".join(map(str, s[0])) + f"-b{s[1]}" for s in SHAPES])
@pytest.mark.parametrize("loss", ["xent", "mse"])
def test_short_batches_of_any_width(B, orc, dims, batch, n, kernels, loss):  # noqa: F811
    check_gradients(B, orc, dims, batch, n, loss, expect=kernels)


@pytest.mark.parametrize("dims,batch,kernels", [([47, 34, 35, 9], 104, {"mlp_thin_forward", "mlp_thin_dgrad", "mlp_wgrad_kernel"}), ([15, 30, 5], 16, {"mlp_thin_forward", "mlp_wgrad_kernel"}),
                                                ([130, 65, 63, 7], 60, {"mlp_thin_forward", "mlp_thin_dgrad", "mlp_wgrad_kernel"}), ([784, 33], 200, {"mlp_thin_forward", "mlp_wgrad_kernel"})])
def test_rows_on_any_boundary(B, orc, dims, batch, kernels):  # noqa: F811
    """Rows without padding, an odd number of parameters: workers and layers start on any 4-byte boundary."""
    assert (sum((a + 1) * b for a, b in zip(dims, dims[1:]))) % 2 == 1
    check_gradients(B, orc, dims, batch, 3, "xent", expect=kernels, pad=1)
