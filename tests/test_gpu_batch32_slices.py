"""Forward products of wide layers on 32 samples, cut along k: workgroups that take two and four slices one after the other, against the oracle."""
import pytest

from test_gpu_grad_mlp import B, check_gradients  # noqa: F401  (B: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,n,forward", [([4096, 128, 10], 9, "fc32_forward"), ([4096, 128, 10], 64, "fc32_forward_2slices"), ([8192, 128, 3], 64, "fc32_forward_4slices")],
                         ids=["one", "two", "four"])
def test_slices_of_a_workgroup(B, orc, dims, n, forward):  # noqa: F811
    check_gradients(B, orc, dims, 32, n, "xent", expect={forward, "fc32_wgrad", "fc_head_kernel"})
