"""Rounds whose gradient kernels form the average on the way (average first, few neighbours): the same bits as a gradient pass and
the averaging kernels, sparse or dense as dbw_mix_path says, which add the same terms in the same order."""
import numpy as np
import pytest
import torch

from paper_2102_06280_amd import inputs
from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2102_06280_amd import binding
    return binding


def hub_graph(n, extra):
    """A ring whose worker 0 is linked to the first `extra` others as well: a list longer than the kernels keep at hand."""
    nb = [set() for _ in range(n)]
    for i in range(n):
        for j in {(i + 1) % n} | ({0} if 0 < i <= extra else set()):
            if i != j:
                nb[i].add(j)
                nb[j].add(i)
    return (np.cumsum([0] + [len(s) for s in nb]).astype(np.int32), np.array([j for s in nb for j in sorted(s)], np.int32))


# dims, batch, loss, workers, pad: one layer in one and in several chunks (aligned and odd rows), batches of at most 16, 32 and 64
# samples with widths that are no multiple of the tiles, long batches with and without split sums, equal widths (the chain)
CASES = [([784, 10], 32, "xent", 8, 64), ([101, 7], 64, "mse", 9, 1), ([257, 16], 300, "xent", 5, 1), ([103, 9], 200, "mse", 13, 64), ([60, 10], 128, "xent", 12, 1), ([300, 9], 40, "xent", 12, 1), ([256, 10], 1024, "xent", 6, 64),
         ([64, 36, 10], 16, "xent", 14, 64), ([300, 92, 10], 32, "mse", 17, 64), ([784, 200, 10], 64, "xent", 24, 64),
         ([100, 36, 52, 3], 50, "xent", 7, 64), ([200, 320, 100, 10], 256, "xent", 14, 64), ([68, 36, 10], 260, "mse", 4, 64),
         ([256, 256, 256, 10], 1024, "mse", 16, 64), ([128, 128, 128, 10], 300, "xent", 12, 64), ([68, 36, 10], 260, "xent", 11, 64), ([784, 200, 10], 64, "xent", 24, 1),
         # widths that are no multiple of four, whose last pairs of rows and groups of columns are moved back: up to 64 samples, steps of 36 and of 32,
         # rows without padding that start on 16-byte boundaries and rows that don't
         ([47, 37, 18, 10], 50, "xent", 20, 64), ([47, 37, 18, 10], 105, "mse", 20, 64), ([47, 37, 18, 10], 109, "xent", 20, 64),
         ([21, 7, 5, 10], 255, "xent", 20, 64), ([617, 301, 75, 26], 101, "xent", 20, 1), ([47, 37, 18, 9], 105, "xent", 20, 1)]


@pytest.mark.parametrize("rates", ["one", "each"])
@pytest.mark.parametrize("dims,batch,loss,n,pad", CASES, ids=["-".join(map(str, c[0])) + f"-b{c[1]}-n{c[3]}-pad{c[4]}" for c in CASES])
def test_average_on_the_way_is_the_average(B, dims, batch, loss, n, pad, rates):
    desc = {"kind": "mlp", "dims": dims, "loss": loss}
    d = inputs.param_count(desc)
    ld = inputs.pad_ld(d, pad)
    rowptr, colidx = hub_graph(n, min(n - 2, 7 if batch <= 32 else 11))       # (the longest lists that are averaged on the way)
    g = np.random.default_rng(77 + n)
    params = inputs.init_params(desc, n, ld, g)
    params[:, :d] += (g.standard_normal((n, d)) * 0.05).astype(np.float32)
    x, y = dev(g.standard_normal((n, batch, dims[0])).astype(np.float32)), dev(g.integers(0, dims[-1], (n, batch)).astype(np.int32))
    t = dev(g.standard_exponential(n).astype(np.float32))
    b = dev(np.minimum(g.integers(0, 2, n), np.diff(rowptr)).astype(np.int32))
    eta = dev(g.uniform(0.01, 0.2, n).astype(np.float32))
    model = B.make_model(B.MODEL_MLP, batch, dims, B.LOSS_MSE if loss == "mse" else B.LOSS_XENT)
    got = {}
    for name in ("way", "pass"):
        h = B.dbw_create(rowptr, colidx, n, d, ld=ld, model=model, mix_path=B.MIX_AUTO if name == "way" else resolved)
        try:
            resolved = B.dbw_mix_path(h)
            out = torch.full((n, ld), 3.0, device="cuda")
            lo = torch.zeros(n, device="cuda")
            B.dbw_select(h, t, b)
            B.dbw_set_timing(h, True)
            if rates == "each":
                B.dbw_round_eta(h, dev(params), out, eta, batch_x=x, batch_y=y, loss_out=lo)
            else:
                B.dbw_round(h, dev(params), out, 0.05, batch_x=x, batch_y=y, loss_out=lo)
            kernels = set(B.dbw_get_timing(h))
            got[name] = (out.cpu().numpy(), lo.cpu().numpy(), any(k.startswith("mix_") for k in kernels))
        finally:
            B.dbw_destroy(h)
    assert got["pass"][2]
    assert got["way"][2] == (ld % 4 != 0 and len(dims) > 2)   # rows off 16-byte boundaries: the kernels that average are not taken
    assert np.array_equal(got["way"][0][:, :d], got["pass"][0][:, :d])
    assert np.all(got["way"][0][:, d:] == 3.0)
    assert np.array_equal(got["way"][1], got["pass"][1])


@pytest.mark.parametrize("dims,batch,extra,on_the_way", [([784, 10], 32, 11, True), ([784, 10], 32, 12, False), ([300, 92, 10], 32, 7, True),
                                                         ([300, 92, 10], 32, 8, False), ([784, 200, 10], 64, 11, True), ([784, 200, 10], 64, 12, False),
                                                         ([256, 256, 256, 10], 256, 15, True), ([256, 256, 256, 10], 256, 16, False), ([256, 10], 300, 30, True)])
def test_long_neighbour_lists_take_the_pass(B, dims, batch, extra, on_the_way):
    """One worker with many neighbours sets the end of the kernels that average on the way, however few the others have on average."""
    n = 32
    rowptr, colidx = hub_graph(n, extra)
    assert np.diff(rowptr).max() == extra + (1 if extra < n - 1 else 0) and colidx.size <= 6 * n
    desc = {"kind": "mlp", "dims": dims, "loss": "xent"}
    d = inputs.param_count(desc)
    ld = inputs.pad_ld(d)
    g = np.random.default_rng(5)
    params = inputs.init_params(desc, n, ld, g)
    x, y = dev(g.standard_normal((n, batch, dims[0])).astype(np.float32)), dev(g.integers(0, dims[-1], (n, batch)).astype(np.int32))
    t, b = dev(g.standard_exponential(n).astype(np.float32)), dev(np.zeros(n, np.int32))
    got = {}
    for mix in (B.MIX_AUTO, B.MIX_CSR):
        h = B.dbw_create(rowptr, colidx, n, d, ld=ld, model=B.make_model(B.MODEL_MLP, batch, dims), mix_path=mix)
        try:
            out = torch.zeros(n, ld, device="cuda")
            B.dbw_select(h, t, b)
            B.dbw_set_timing(h, True)
            B.dbw_round(h, dev(params), out, 0.05, batch_x=x, batch_y=y)
            got[mix] = (out.cpu().numpy(), any(k.startswith("mix_") for k in B.dbw_get_timing(h)))
        finally:
            B.dbw_destroy(h)
    assert got[B.MIX_CSR][1] and got[B.MIX_AUTO][1] != on_the_way
    assert np.array_equal(got[B.MIX_AUTO][0], got[B.MIX_CSR][0])


@pytest.mark.parametrize("dims,batch,n,degree,on_the_way", [([784, 36, 10], 64, 37, 2, True), ([784, 36, 10], 64, 37, 4, False), ([784, 36, 10], 16, 40, 4, False),
                                                            ([784, 36, 10], 32, 40, 4, True), ([784, 36, 10], 32, 40, 6, False), ([784, 100, 10], 8, 56, 6, True),
                                                            ([256, 384, 10], 256, 24, 4, True), ([256, 384, 10], 256, 24, 6, False), ([128, 384, 10], 256, 30, 6, True),
                                                            ([784, 10], 8, 128, 4, True), ([784, 10], 8, 128, 6, False),
                                                            ([784, 10], 8, 192, 2, False), ([784, 10], 70, 192, 2, True), ([64, 36, 10], 16, 7, 4, True),
                                                            ([64, 36, 10], 16, 8, 4, False), ([64, 36, 10], 32, 9, 4, True), ([784, 384, 200, 10], 256, 12, 4, False), ([256, 256, 256, 10], 300, 12, 4, True),
                                                            ([300, 37, 10], 100, 40, 6, True), ([300, 37, 10], 100, 40, 8, False), ([1024, 255, 10], 96, 64, 6, True)])
def test_many_neighbours_take_the_pass(B, dims, batch, n, degree, on_the_way):
    """Every worker linked to the nearest `degree` on a circle: how many the kernels average on the way depends on the tiles of the gradients."""
    nb = [sorted({(i + k) % n for k in range(-(degree // 2), degree // 2 + 1)} - {i}) for i in range(n)]
    rowptr, colidx = np.cumsum([0] + [len(s) for s in nb]).astype(np.int32), np.array(sum(nb, []), np.int32)
    d = inputs.param_count({"kind": "mlp", "dims": dims, "loss": "xent"})
    ld = inputs.pad_ld(d)
    g = np.random.default_rng(6)
    params = inputs.init_params({"kind": "mlp", "dims": dims, "loss": "xent"}, n, ld, g)
    x, y = dev(g.standard_normal((n, batch, dims[0])).astype(np.float32)), dev(g.integers(0, dims[-1], (n, batch)).astype(np.int32))
    t, b = dev(g.standard_exponential(n).astype(np.float32)), dev(np.ones(n, np.int32))
    got, resolved = {}, B.MIX_AUTO
    for name in ("auto", "pass"):
        h = B.dbw_create(rowptr, colidx, n, d, ld=ld, model=B.make_model(B.MODEL_MLP, batch, dims), mix_path=resolved)
        try:
            resolved = B.dbw_mix_path(h)
            out = torch.zeros(n, ld, device="cuda")
            B.dbw_select(h, t, b)
            B.dbw_set_timing(h, True)
            B.dbw_round(h, dev(params), out, 0.05, batch_x=x, batch_y=y)
            got[name] = (out.cpu().numpy(), any(k.startswith("mix_") for k in B.dbw_get_timing(h)))
        finally:
            B.dbw_destroy(h)
    assert got["pass"][1] and got["auto"][1] != on_the_way
    assert np.array_equal(got["auto"][0], got["pass"][0])


@pytest.mark.parametrize("what", ["batch_x", "batch_y", "loss_out"])
def test_buffers_inside_the_new_parameters_take_the_pass(B, what):
    """The batch may lie where the new parameters go, and the losses may lie there: all gradients are taken before anything is written."""
    dims, batch, n = [256, 36, 10], 4, 16
    rowptr, colidx = hub_graph(n, 3)
    desc = {"kind": "mlp", "dims": dims, "loss": "xent"}
    d = inputs.param_count(desc)
    ld = inputs.pad_ld(d)
    g = np.random.default_rng(6)
    params = dev(inputs.init_params(desc, n, ld, g))
    x, y = dev(g.standard_normal((n, batch, dims[0])).astype(np.float32)), dev(g.integers(0, dims[-1], (n, batch)).astype(np.int32))
    t, b = dev(g.standard_exponential(n).astype(np.float32)), dev(np.zeros(n, np.int32))
    h = B.dbw_create(rowptr, colidx, n, d, ld=ld, model=B.make_model(B.MODEL_MLP, batch, dims))
    try:
        got = []
        for inside in (False, True):
            out, loss, bx, by = torch.zeros(n, ld, device="cuda"), torch.zeros(n, device="cuda"), x, y
            if inside and what == "batch_x":
                bx = out.view(-1)[64:64 + x.numel()].view(x.shape)
                bx.copy_(x)
            elif inside and what == "batch_y":
                by = out.view(-1)[3 * ld:3 * ld + y.numel()].view(y.shape).view(torch.int32)
                by.copy_(y)
            elif inside:
                loss = out.view(-1)[5 * ld + 8:5 * ld + 8 + n]
            B.dbw_select(h, t, b)
            B.dbw_set_timing(h, True)
            B.dbw_round(h, params, out, 0.05, batch_x=bx, batch_y=by, loss_out=loss)
            assert any(k.startswith("mix_") for k in B.dbw_get_timing(h)) == inside
            B.dbw_set_timing(h, False)
            got.append(out[:, :d].cpu().numpy())
        assert np.array_equal(got[0], got[1])
    finally:
        B.dbw_destroy(h)


@pytest.mark.parametrize("dims,batch", [([784, 10], 32), ([256, 10], 300), ([100, 36, 10], 24), ([64, 36, 10], 260)])
@pytest.mark.parametrize("n,degree,path", [(6, 2, "dense"), (9, 4, "dense"), (10, 4, "dense"), (16, 2, "sparse")])
def test_diverged_worker_reaches_the_rows_that_the_path_says(B, dims, batch, n, degree, path):
    """A NaN and an infinity in the parameters of a worker that nobody waits for: in every row of a dense average, in its own row alone of
    a sparse one, wherever the new parameters lie."""
    g = np.random.default_rng(n)
    rowptr, colidx = inputs.graph_ring(n) if degree == 2 else inputs.graph_regular(n, degree, g)
    desc = {"kind": "mlp", "dims": dims, "loss": "xent"}
    d = inputs.param_count(desc)
    ld = inputs.pad_ld(d)
    params = inputs.init_params(desc, n, ld, g)
    params[3, d - 2], params[3, 5] = np.nan, np.inf
    params = dev(params)
    x, y = dev(g.standard_normal((n, batch, dims[0])).astype(np.float32)), dev(g.integers(0, dims[-1], (n, batch)).astype(np.int32))
    times = g.standard_exponential(n).astype(np.float32)
    times[3] = 100.0
    b = np.where([3 in colidx[rowptr[i]:rowptr[i + 1]] for i in range(n)], 1, 0).astype(np.int32)
    h = B.dbw_create(rowptr, colidx, n, d, ld=ld, model=B.make_model(B.MODEL_MLP, batch, dims))
    try:
        assert B.dbw_mix_path(h) == (B.MIX_DENSE if path == "dense" else B.MIX_CSR)
        got = []
        for shift in (0, 1):                            # new parameters on a 16-byte boundary and off it
            out = torch.zeros(n * ld + 1, device="cuda")[shift:shift + n * ld].view(n, ld)
            B.dbw_select(h, dev(times), dev(b))
            B.dbw_round(h, params, out, 0.05, batch_x=x, batch_y=y)
            got.append(out[:, :d].cpu().numpy())
    finally:
        B.dbw_destroy(h)
    others = np.arange(n) != 3
    for o in got:
        assert np.all(np.isnan(o[3]))                   # (its gradient is NaN throughout)
        reached = ~np.isfinite(o[others])
        assert np.array_equal(reached.sum(1), np.full(n - 1, 2 if path == "dense" else 0))
        if path == "dense":
            assert np.all(np.isnan(o[others][:, d - 2])) and np.all(np.isnan(o[others][:, 5]))
    assert np.array_equal(got[0], got[1], equal_nan=True)
