"""Gradients of networks whose second layer has few channels, against the oracle: up to sixteen output channels, of the forward pass
(channels 2) or of the data gradient (channels 1), take matrix instructions of two taps a step, of which the last one's second is none; more take
one tap.  Channels on both sides of the line, more input channels than one group of sixteen, windows that fill no block; the last two have the weight gradient's workgroups two to a compute unit."""
import numpy as np
import pytest
import torch

from paper_2102_06280_amd import inputs
from gpu_util import GradientResolver, dev, match_gradients
from test_gpu_grad_cnn import B, cnn_desc, layers_close  # noqa: F401  (B: the fixture)

pytestmark = pytest.mark.gpu

# input channels, height, width, channels 1 and 2, filter, dense, classes; batch
SHAPES = [((1, 8, 8, 16, 16, 3, 6, 5), 17), ((1, 28, 28, 15, 17, 5, 6, 5), 3), ((2, 12, 20, 17, 15, 3, 6, 5), 4), ((1, 16, 16, 1, 2, 5, 6, 5), 5),
          ((3, 20, 12, 33, 16, 5, 7, 4), 3), ((1, 12, 12, 16, 40, 3, 6, 5), 6), ((1, 8, 8, 7, 4, 5, 6, 5), 150), ((1, 8, 8, 13, 33, 5, 6, 5), 120)]


@pytest.mark.parametrize("shape,batch", SHAPES, ids=["-".join(map(str, s[0])) + f"-b{s[1]}" for s in SHAPES])
def test_second_layer_matches_oracle(B, orc, shape, batch):  # noqa: F811
    n, g, desc = 3, np.random.default_rng(700 + shape[3]), cnn_desc(shape)
    d = inputs.param_count(desc)
    ld = inputs.pad_ld(d)
    rowptr, colidx = inputs.graph_ring(n)
    params = inputs.init_params(desc, n, ld, g)
    params[:, :d] += (g.standard_normal((n, d)) * 0.02).astype(np.float32)
    x = g.standard_normal((n, batch, shape[0] * shape[1] * shape[2])).astype(np.float32)
    y = g.integers(0, shape[-1], (n, batch)).astype(np.int32)
    h = B.dbw_create(rowptr, colidx, n, d, ld=ld, model=B.make_model(B.MODEL_CNN, batch, shape))
    try:
        grads = torch.full((n, ld), 7.0, dtype=torch.float32, device="cuda")
        loss = torch.zeros(n, dtype=torch.float32, device="cuda")
        B.dbw_grad(h, dev(params), dev(x), dev(y), grads, loss)
        got = grads.cpu().numpy()
        kind, od = orc.model_desc(desc)
        res = GradientResolver(orc, kind, od, d, params, x, y, threads=n)
        assert np.allclose(loss.cpu().numpy(), res.loss, rtol=5e-6, atol=1e-6)
        assert np.all(got[:, d:] == 7.0)
        match_gradients(res, got, layers_close(desc), d, what=str(shape))
    finally:
        B.dbw_destroy(h)
