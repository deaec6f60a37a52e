"""Rounding of the gradients against 64 bits, layer by layer, where a sum over the batch can be formed in one piece or in several: long
chunks of samples in the fused head, up to 32 classes, batches of 65 to 255 samples, last layers whose width is no multiple of four.

Bounds: the median over the workers of the relative error (2-norm) that the batched GEMM kernels and a head on chunks of 16 samples have on
these inputs, in units of 1e-7, times 1.03.  The inputs are seeded and the sums have a fixed order, so the errors are the same in every run."""
import numpy as np
import pytest
import torch

from paper_2102_06280_amd import inputs

pytestmark = pytest.mark.gpu

# dims, batch, workers, loss, seeds, {gradient: error with those kernels}
CASES = [([784, 10], 150, 30, "xent", 3, {"dW1": 1.29, "db1": 1.37}), ([200, 10], 300, 60, "xent", 1, {"dW1": 1.19, "db1": 1.56}),
         ([256, 25], 1024, 8, "xent", 6, {"dW1": 1.43, "db1": 1.99}), ([301, 32], 64, 32, "xent", 3, {"dW1": 1.47, "db1": 1.55}),
         ([64, 33], 200, 16, "xent", 6, {"dW1": 1.38, "db1": 1.41}), ([784, 200, 10], 128, 32, "xent", 3, {"dW2": 2.27, "dW1": 1.84}),
         ([784, 300, 10], 200, 32, "xent", 3, {"dW2": 3.22, "dW1": 2.89}), ([64, 48, 25], 300, 32, "xent", 3, {"dW2": 1.24, "dW1": 1.19, "db1": 0.72}),
         ([128, 96, 20], 1024, 16, "xent", 6, {"dW2": 1.13, "db2": 0.64, "dW1": 1.90, "db1": 0.65})]


def errors(B, dims, batch, n, loss, seed, out):
    g = np.random.default_rng(seed)
    desc = {"kind": "mlp", "dims": dims, "loss": loss}
    d = inputs.param_count(desc)
    ld = inputs.pad_ld(d)
    params = inputs.init_params(desc, n, ld, g)
    params[:, :d] += (g.standard_normal((n, d)) * 0.02).astype(np.float32)
    x = torch.from_numpy(g.standard_normal((n, batch, dims[0])).astype(np.float32)).cuda()
    y = torch.from_numpy(g.integers(0, dims[-1], (n, batch)).astype(np.int32)).cuda()
    p = torch.from_numpy(params).cuda()
    grads = torch.zeros((n, ld), device="cuda")
    h = B.dbw_create(*inputs.graph_ring(n), n, d, ld=ld, model=B.make_model(B.MODEL_MLP, batch, dims, B.LOSS_XENT))
    try:
        B.dbw_grad(h, p, x, y, grads, torch.zeros(n, device="cuda"))
        torch.cuda.synchronize()
    finally:
        B.dbw_destroy(h)
    at = [0]
    for fan_in, nw, nb in inputs.layer_shapes(desc):
        at += [at[-1] + nw, at[-1] + nw + nb]
    L = len(dims) - 1
    for w in range(n):
        row, got = p[w].double(), grads[w].double()
        weights = [row[at[2 * l]:at[2 * l + 1]].view(dims[l + 1], dims[l]) for l in range(L)]
        a = [x[w].double()]
        for l in range(L):
            z = a[-1] @ weights[l].t() + row[at[2 * l + 1]:at[2 * l + 2]]
            a.append(z if l == L - 1 else z.relu())
        dz = (torch.softmax(a[-1], 1) - torch.nn.functional.one_hot(y[w].long(), dims[-1]).double()) / batch
        for l in reversed(range(L)):
            for name, want, lo in ((f"dW{l + 1}", (dz.t() @ a[l]).flatten(), at[2 * l]), (f"db{l + 1}", dz.sum(0), at[2 * l + 1])):
                e = (got[lo:lo + want.numel()] - want).norm() / want.norm()
                out.setdefault(name, []).append(e.item())
            dz = (dz @ weights[l]) * (a[l] > 0)


@pytest.mark.parametrize("dims,batch,n,loss,seeds,bounds", CASES, ids=["-".join(map(str, c[0])) + f"-b{c[1]}" for c in CASES])
def test_sums_over_the_batch(dims, batch, n, loss, seeds, bounds):
    from paper_2102_06280_amd import binding as B
    out = {}
    for seed in range(seeds):
        errors(B, dims, batch, n, loss, 7 + seed, out)
    got = {k: 1e7 * float(np.median(v)) for k, v in out.items()}
    print({k: round(v, 3) for k, v in got.items()})
    assert all(got[k] <= 1.03 * bound for k, bound in bounds.items()), (got, bounds)
