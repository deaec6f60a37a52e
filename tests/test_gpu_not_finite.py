"""Infinities, NaN and the largest floats in the kernels that split fp32 values into three bf16 values: element by element
what plain sums give (the oracle), and in about the time that other values take."""
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


def same_elements(got, want, slices, tol):
    """NaN and infinities where the oracle has them, and nowhere else; the finite rest of every layer within tol of its
    largest element and norm (or 1e-7: the deltas, up to 1 / batch and rounded to 2^-24 of that, can cancel in a bias gradient)."""
    for lo, hi in slices:
        g, w = got[lo:hi].astype(np.float64), want[lo:hi].astype(np.float64)
        for what, f in (("NaN", np.isnan), ("+inf", np.isposinf), ("-inf", np.isneginf)):
            assert np.array_equal(f(g), f(w)), f"[{lo}:{hi}] {what}: {f(g).sum()} here, {f(w).sum()} in the oracle"
        ok = np.isfinite(w)
        if ok.any():
            diff, size = g[ok] - w[ok], np.abs(w[ok]).max()
            assert np.abs(diff).max() <= max(tol * size, 1e-7), f"[{lo}:{hi}]"
            assert np.linalg.norm(diff) <= max(tol * np.linalg.norm(w[ok]), 1e-7), f"[{lo}:{hi}]"


def slices_of(desc):
    off, out = 0, []
    for _, nw, nb in inputs.layer_shapes(desc):
        out += [(off, off + nw), (off + nw, off + nw + nb)]
        off += nw + nb
    return out


def gradients(B, desc, dims, params, x, y):
    n, batch = x.shape[:2]
    d = inputs.param_count(desc)
    rowptr, colidx = inputs.graph_complete(n)
    kind = B.MODEL_CNN if desc["kind"] == "cnn" else B.MODEL_MLP
    h = B.dbw_create(rowptr, colidx, n, d, ld=params.shape[1], model=B.make_model(kind, batch, dims))
    try:
        grads, loss = torch.zeros(params.shape, device="cuda"), torch.zeros(n, device="cuda")
        B.dbw_grad(h, dev(params), dev(x), dev(y), grads, loss)
        return grads.cpu().numpy()[:, :d], loss.cpu().numpy()
    finally:
        B.dbw_destroy(h)


# One filter row and two with a partial last step, widths on and off 16 and 8, 3 x 3 and 5 x 5, one and several blocks of
# output channels, one and several samples per workgroup, shared blocks of the weight gradient and not.
CNN = [(1, 28, 28, 6, 16, 5, 20, 10), (3, 12, 20, 9, 40, 5, 12, 5), (2, 16, 16, 17, 33, 3, 12, 4), (1, 8, 8, 4, 70, 3, 8, 3)]
CNN_WHERE = ["pixels", "pooled", "largest", "conv1 +inf", "conv2 +inf", "conv2 -inf", "conv2 nan"]


@pytest.mark.parametrize("where", CNN_WHERE)
@pytest.mark.parametrize("shape", CNN, ids=["-".join(map(str, s)) for s in CNN])
def test_cnn_element_by_element(B, orc, shape, where):
    """Worker 1 of two, batch 3.  pixels: an infinite pixel inside one sample and one in the corner of another, under negative
    filters, so that the pooled maps and the loss stay finite and only those weight gradients of conv1 are lost that the
    pixels enter (0 * inf), not those of filter positions that would need an output outside the image.  pooled: an infinite pixel under
    positive filters of one channel, whose pooled values conv2 multiplies by negative weights only, so that every delta that meets them
    is zero and all other sums are finite: conv2's weight gradient of that channel is lost (0 * inf), of the others none.  largest: the
    largest float as a pixel.  conv1 / conv2: one infinite or NaN weight at a filter's centre, which no output reaches
    over the border with; conv1's under positive pixels, so that the channel is infinite throughout, and below filters
    of both signs, so that all of conv2 is inf - inf.  Tolerance as for finite gradients (3e-5 per layer)."""
    C0, H, W, C1, C2, K, F, NC = shape
    desc = {"kind": "cnn", "in": (C0, H, W), "c1": C1, "c2": C2, "k": K, "fc": F, "classes": NC}
    d, KK = inputs.param_count(desc), K * K
    g = np.random.default_rng(11)
    params = inputs.init_params(desc, 2, d + 3, g)
    x = g.standard_normal((2, 3, C0, H, W)).astype(np.float32)
    y = g.integers(0, NC, (2, 3)).astype(np.int32)
    c, centre = C0 - 1, KK // 2
    w1 = params[1, :C1 * C0 * KK].reshape(C1, C0, KK)
    b1 = params[:, C1 * C0 * KK:C1 * C0 * KK + C1]
    w2 = params[1, C1 * C0 * KK + C1:][:C2 * C1 * KK].reshape(C2, C1, KK)
    if where == "pixels":
        w1[:, c] = -np.abs(w1[:, c]) - 0.01
        x[1, 0, c, H // 2, W // 2] = np.inf
        x[1, 2, c, 0, W - 1] = np.inf
    elif where == "pooled":
        w1[:, c] = -np.abs(w1[:, c]) - 0.01
        w1[C1 - 1, c] *= -1.0
        w2[:, C1 - 1] = -np.abs(w2[:, C1 - 1]) - 0.01
        x[1, 0, c, H // 2, W // 2] = np.inf
    elif where == "largest":
        params[1, :C1 * C0 * KK] *= 1e-6
        x[1, 0, c, H // 2, W // 2] = np.finfo(np.float32).max
    elif where == "conv1 +inf":
        x[1, :, c] = np.abs(x[1, :, c]) + 0.1
        w1[C1 - 1, c, centre] = np.inf
        w2[:, C1 - 1] = np.abs(w2[:, C1 - 1]) * (-1.0) ** np.arange(KK)
    else:
        b1[:] = 10.0                                    # every pooled value of the first layer is positive
        w2[C2 - 1, C1 - 1, centre] = float(where.split()[1])
    x = x.reshape(2, 3, -1)
    got, loss = gradients(B, desc, shape, params, x, y)
    kind, od = orc.model_desc(desc)
    want, wloss = orc.grad_all(kind, od, d, params, x, y)[:2]
    if where == "pixels":
        lost = np.isnan(want[1, :C1 * C0 * KK].reshape(C1, C0, KK))
        assert lost[:, c].all() and not lost[:, :c].any() and np.isfinite(want[1, C1 * C0 * KK:d]).all()
    if where == "pooled":
        lost = np.isnan(want[1, C1 * C0 * KK + C1:][:C2 * C1 * KK].reshape(C2, C1, KK))
        assert lost[:, C1 - 1].any(1).all() and not lost[:, :C1 - 1].any() and np.isfinite(want[1, C1 * C0 * KK + C1 + C2 * C1 * KK:d]).all()
    np.testing.assert_allclose(loss, wloss, rtol=5e-6, atol=1e-6)
    for i in range(2):
        same_elements(got[i], want[i, :d], slices_of(desc), 3e-5)


def test_corner_pixel_reaches_its_own_taps_only(B, orc):
    """An infinite pixel in the upper right corner, alone: the weight gradients of the filter positions that no output inside the
    image pairs with it stay finite and right, on a width that is padded to a multiple of 16 in the kernel."""
    shape = (1, 12, 20, 9, 8, 5, 12, 5)
    desc = {"kind": "cnn", "in": shape[:3], "c1": 9, "c2": 8, "k": 5, "fc": 12, "classes": 5}
    d = inputs.param_count(desc)
    g = np.random.default_rng(12)
    params = inputs.init_params(desc, 2, d, g)
    params[:, :9 * 25] = -np.abs(params[:, :9 * 25]) - 0.01
    params[:, 9 * 25:9 * 25 + 9] = 0.5
    x = g.standard_normal((2, 3, 12, 20)).astype(np.float32)
    x[1, 1, 0, 19] = np.inf
    x = x.reshape(2, 3, -1)
    y = g.integers(0, 5, (2, 3)).astype(np.int32)
    got, _ = gradients(B, desc, shape, params, x, y)
    kind, od = orc.model_desc(desc)
    want = orc.grad_all(kind, od, d, params, x, y)[0]
    lost = np.isnan(want[1, :9 * 25].reshape(9, 5, 5))
    assert lost[:, :3, 2:].all() and lost.sum() == 9 * 9
    for i in range(2):
        same_elements(got[i], want[i, :d], slices_of(desc), 3e-5)


@pytest.mark.parametrize("sign", [-1, 1])
@pytest.mark.parametrize("dims,batch", [([65, 63, 70, 20], 66), ([129, 64, 33, 18], 65), ([7, 9, 21], 130),
                                        ([65, 63, 70, 40], 266), ([129, 64, 33, 34], 257), ([7, 9, 37], 300)], ids=["65", "129", "7", "65-long", "129-long", "7-long"])
def test_mlp_element_by_element(B, orc, dims, batch, sign):
    """An infinite input value of worker 1 under first-layer weights of one sign.  Negative: the layer is -inf, after ReLU zero,
    and of the gradients only that input's column is lost (0 * inf).  Positive: the activations are infinite and the layer above gets
    inf - inf, so with a third layer its weight gradient is lost as well (0 * inf), with two layers everything is.  Batches of up to 255 take
    the fp32 kernels and up to 32 classes the fused head, longer batches of odd widths and more classes the split products."""
    desc = {"kind": "mlp", "dims": dims, "loss": "xent"}
    d = inputs.param_count(desc)
    g = np.random.default_rng(21)
    params = inputs.init_params(desc, 3, d, g)
    x = g.standard_normal((3, batch, dims[0])).astype(np.float32)
    y = g.integers(0, dims[-1], (3, batch)).astype(np.int32)
    x[1, 4, 3] = np.inf
    w = params[1, :dims[0] * dims[1]].reshape(dims[1], dims[0])
    w[:, 3] = sign * (np.abs(w[:, 3]) + 0.01)
    got, loss = gradients(B, desc, dims, params, x, y)
    kind, od = orc.model_desc(desc)
    want, wloss = orc.grad_all(kind, od, d, params, x, y)[:2]
    np.testing.assert_allclose(loss, wloss, rtol=5e-6, atol=1e-6)
    if sign < 0:
        assert np.isnan(want[1, :d]).sum() == dims[1]
    for i in range(3):
        same_elements(got[i], want[i, :d], slices_of(desc), 2e-5)


def _time(fn):
    best = float("inf")
    for _ in range(4):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        fn()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("model", ["dense average", "perceptron", "convolutions"])
def test_time_with_values_that_are_not_finite(B, model):
    """A worker that has diverged must not hold up the others: with NaN or infinities throughout one worker's parameters, or a
    single one of either, a call takes at most three times as long as with finite values (a kernel that goes through its
    products a second and a third time; lane-by-lane sums took 13 to 75 times as long)."""
    n = 64 if model == "dense average" else 8
    rowptr, colidx = inputs.graph_complete(n)
    if model == "dense average":
        d, desc, kw = 400_000, None, {"mix_path": B.MIX_DENSE}
    else:
        if model == "perceptron":
            dims, batch = [256, 395, 295, 64, 28], 1024
            desc, kind = {"kind": "mlp", "dims": dims, "loss": "xent"}, B.MODEL_MLP
        else:
            dims, batch = [3, 32, 32, 32, 64, 5, 64, 10], 32
            desc, kind = {"kind": "cnn", "in": (3, 32, 32), "c1": 32, "c2": 64, "k": 5, "fc": 64, "classes": 10}, B.MODEL_CNN
        d, kw = inputs.param_count(desc), {"model": B.make_model(kind, batch, dims)}
    ld = inputs.pad_ld(d)
    g = np.random.default_rng(31)
    x = dev(inputs.init_params(desc, n, ld, g) if desc else g.standard_normal((n, ld)).astype(np.float32))
    out = torch.zeros_like(x)
    h = B.dbw_create(rowptr, colidx, n, d, ld=ld, **kw)
    try:
        if desc is None:
            B.dbw_select(h, dev(g.standard_exponential(n).astype(np.float32)), dev(np.full(n, 5, np.int32)))
            def call(): B.dbw_round(h, x, out, 0.0)
        else:
            bx = dev(g.standard_normal((n, batch, 256 if model == "perceptron" else 3 * 32 * 32)).astype(np.float32))
            by, loss = dev(g.integers(0, 10, (n, batch)).astype(np.int32)), torch.zeros(n, device="cuda")
            def call(): B.dbw_grad(h, x, bx, by, out, loss)
        finite, values = _time(call), x.clone()
        for v in (float("nan"), float("inf")):
            for whole in (True, False):
                x.copy_(values)
                if whole:
                    x[1] = v
                else:
                    x[1, 100] = v
                t = _time(call)
                assert t <= 3 * finite, f"{v} {'throughout' if whole else 'once'}: {t:.3f} ms, finite {finite:.3f}"
    finally:
        B.dbw_destroy(h)
