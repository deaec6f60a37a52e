"""Gradients of networks whose first layer has one to seven input channels, against the oracle: every phase of the reduction over
filter rows and taps (rows of either half of a wavefront, one period of eight rows and more), narrow and ragged images, more than
one block of output channels."""
import numpy as np
import pytest
import torch

from paper_2102_06280_amd import inputs
from gpu_util import GradientResolver, dev, match_gradients
from test_gpu_grad_cnn import B, cnn_desc, layers_close  # noqa: F401  (B: the fixture)

pytestmark = pytest.mark.gpu

# input channels, height, width, channels 1 and 2, filter, dense, classes; batch
SHAPES = [((1, 8, 8, 4, 3, 3, 6, 5), 5), ((1, 12, 28, 16, 4, 5, 6, 5), 3), ((2, 12, 8, 9, 4, 5, 6, 5), 4), ((2, 16, 16, 32, 4, 3, 6, 5), 3),
          ((3, 20, 20, 12, 3, 3, 7, 4), 3), ((3, 32, 32, 32, 3, 5, 6, 5), 2), ((4, 8, 12, 16, 4, 3, 6, 5), 9), ((4, 16, 12, 17, 4, 5, 6, 5), 2),
          ((5, 8, 20, 33, 3, 3, 6, 5), 4), ((6, 12, 12, 5, 4, 5, 6, 5), 3), ((7, 8, 8, 40, 3, 3, 6, 5), 2),
          ((6, 8, 12, 17, 3, 3, 6, 5), 4), ((6, 12, 8, 16, 3, 3, 6, 5), 4), ((8, 16, 16, 9, 3, 3, 6, 5), 3), ((3, 12, 48, 5, 3, 5, 6, 5), 2)]


def check_gradients(B, orc, shape, batch, n):  # noqa: F811
    g, desc = np.random.default_rng(900 + shape[0]), cnn_desc(shape)
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


@pytest.mark.parametrize("shape,batch", SHAPES, ids=["-".join(map(str, s[0])) + f"-b{s[1]}" for s in SHAPES])
def test_first_layer_matches_oracle(B, orc, shape, batch):  # noqa: F811
    check_gradients(B, orc, shape, batch, 3)


# 8 workers: the first layer's weight gradient takes two (the fifth shape: three) samples to a workgroup, with one and two blocks of output
# channels and both filter sizes, the second's three, three, two, two, seven and three, with 5 x 5 filters also as two workgroups to a compute
# unit; the last workgroup of a worker has fewer.
SHARED = [((1, 8, 8, 12, 3, 3, 6, 5), 161), ((3, 8, 8, 9, 3, 5, 6, 5), 161), ((2, 8, 8, 20, 35, 3, 6, 5), 115), ((3, 8, 8, 24, 4, 5, 6, 5), 115),
          ((1, 8, 8, 33, 100, 5, 6, 5), 97), ((3, 20, 20, 9, 3, 5, 6, 5), 161)]


@pytest.mark.parametrize("shape,batch", SHARED, ids=["-".join(map(str, s[0])) + f"-b{s[1]}" for s in SHARED])
def test_workgroups_of_several_samples_match_oracle(B, orc, shape, batch):  # noqa: F811
    check_gradients(B, orc, shape, batch, 8)


def test_weight_gradient_sums_are_as_exact_as_fp32_ones(B):  # noqa: F811
    """3 -> 32 channels on 32 x 32 pixels, 5 x 5, 64 workers x 32 samples: three samples to a workgroup.  Filters of one and two taps, saturated
    logits and hidden units that are always on make everything before and behind conv1's weight gradient exact, so that its error is that of
    its sums.  fp32 multiply-adds of 512 pixels, one in fifteen of which has a delta, and the addition of 64 such sums, each rounding 2.4e-8
    of the sum so far in the root mean square: 2.4e-8 (34 / 2 + 64 / 2)^(1/2) = 1.7e-7 of the result."""
    import torch.nn.functional as F
    n, batch, shape = 64, 32, (3, 32, 32, 32, 64, 5, 512, 10)
    desc = cnn_desc(shape)
    d = inputs.param_count(desc)
    ld = inputs.pad_ld(d)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(77)

    def integers(lo, hi, size):                         # lo .. hi
        return torch.randint(lo, hi + 1, size, device="cuda", generator=gen).float()

    def taps(size, count, values):
        at = torch.rand(size, device="cuda", generator=gen).argsort(dim=-1)[..., :count]
        return torch.zeros(size, device="cuda").scatter_(-1, at, values)

    parts = [taps((n, 32, 75), 2, integers(0, 1, (n, 32, 2)) * 2 - 1), integers(-2, 2, (n, 32)) / 4, taps((n, 64, 800), 1, torch.ones(n, 64, 1, device="cuda")),
             torch.zeros(n, 64, device="cuda"), integers(-255, 255, (n, 512, 4096)) * (integers(0, 15, (n, 512, 4096)) == 0) * 2.0 ** -30,
             torch.ones(n, 512, device="cuda"), integers(-8, 8, (n, 10, 512)) / 8, torch.zeros(n, 10, device="cuda")]
    parts[7][:, 3] = 4096.0
    params = torch.zeros(n, ld, device="cuda")
    params[:, :d] = torch.cat([p.flatten(1) for p in parts], 1)
    x = integers(-2 ** 21, 2 ** 21 - 1, (n, batch, 3 * 32 * 32)) * 2.0 ** -20
    y = (4 + torch.randint(0, 6, (n, batch), device="cuda", generator=gen)).int()
    rowptr, colidx = inputs.graph_ring(n)
    h = B.dbw_create(rowptr, colidx, n, d, ld=ld, model=B.make_model(B.MODEL_CNN, batch, shape))
    try:
        grads = torch.zeros_like(params)
        B.dbw_grad(h, params, x, y, grads, torch.zeros(n, device="cuda"))
    finally:
        B.dbw_destroy(h)
    error = total = 0.0
    for i in range(0, n, 8):                            # every eighth worker in 64 bits
        w1 = parts[0][i].double().requires_grad_(True)
        cols = F.unfold(x[i].double().view(batch, 3, 32, 32), 5, padding=2).transpose(1, 2).reshape(-1, 75)
        z = (cols @ w1.t() + parts[1][i].double()).view(batch, 1024, 32).transpose(1, 2).reshape(batch, 32, 32, 32)
        a = F.max_pool2d(torch.relu(z), 2)
        cols = F.unfold(a, 5, padding=2).transpose(1, 2).reshape(-1, 800)
        z = (cols @ parts[2][i].double().t()).view(batch, 256, 64).transpose(1, 2).reshape(batch, 64, 16, 16)
        a = F.max_pool2d(torch.relu(z), 2).flatten(1)
        a = torch.relu(a @ parts[4][i].double().t() + 1.0)
        assert float(a.detach().min()) > 0
        loss = F.cross_entropy(a @ parts[6][i].double().t() + parts[7][i].double(), y[i].long())
        want = torch.autograd.grad(loss, w1)[0]
        got = grads[i, :want.numel()].view_as(want).double()
        error += float((got - want).square().sum())
        total += float(want.square().sum())
    assert (error / total) ** 0.5 < 1.7e-7
