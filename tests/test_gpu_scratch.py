"""Device memory of a context: no partial sums of the fused head for a last layer that the head does not take."""
import pytest
import torch

from paper_2102_06280_amd import inputs

pytestmark = pytest.mark.gpu


def context_bytes(B, dims, batch, n):
    rowptr, colidx = inputs.graph_ring(n)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    h = B.dbw_create(rowptr, colidx, n, inputs.param_count({"kind": "mlp", "dims": dims, "loss": "xent"}), model=B.make_model(B.MODEL_MLP, batch, dims))
    used = free - torch.cuda.mem_get_info()[0]
    B.dbw_destroy(h)
    return used


@pytest.mark.parametrize("classes", [10, 20, 32, 33])
def test_wide_inputs_of_a_single_layer(classes):
    """100 000 inputs don't fit the head's LDS.  A context holds the workers' gradients and, of their split products, the logits: 58 MB with 33
    classes; partial sums of W for every 16 samples would be 32 times the gradients."""
    from paper_2102_06280_amd import binding as B
    n, batch, inputs_ = 4, 512, 100_000
    B.dbw_destroy(B.dbw_create(*inputs.graph_ring(n), n, 64))            # whatever the first context brings with it
    parameters = 4 * n * classes * (inputs_ + 1)
    scratch = 4 * n * batch * classes * (2 + 16)
    assert context_bytes(B, [inputs_, classes], batch, n) <= parameters + scratch + (32 << 20)
