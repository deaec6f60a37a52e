"""Averages whose workgroups take more than one round of column tiles, the last one partial: every column, on rows with and without
padding, sparse and dense, against the weight matrix times the parameters in 64 bits."""
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


# workers, columns, dense; tiles of 256, 128 and 64 columns (sparse), of 64, 64 and 32 (dense), on 256 or 512 workgroups
@pytest.mark.parametrize("order", ["cta", "atc"])
@pytest.mark.parametrize("pad", [64, 1])
@pytest.mark.parametrize("n,d,dense", [(48, 256 * 256 + 700, False), (48, 256 * 700 + 3, False), (128, 128 * 300 + 5, False), (256, 64 * 257 + 1, False),
                                       (40, 64 * 513 + 7, True), (40, 64 * 1100, True), (128, 64 * 260 + 9, True), (256, 32 * 520 + 1, True)])
def test_every_column_once(B, n, d, dense, pad, order):
    g = np.random.default_rng(n + d)
    rowptr, colidx = inputs.graph_complete(n) if dense else inputs.graph_regular(n, 4, g)
    ld = inputs.pad_ld(d, pad)
    x = g.standard_normal((n, ld)).astype(np.float32)
    gr = (g.standard_normal((n, ld)) * 0.1).astype(np.float32)
    h = B.dbw_create(rowptr, colidx, n, d, ld=ld, mix_path=B.MIX_DENSE if dense else B.MIX_CSR, order=B.ORDER_ATC if order == "atc" else B.ORDER_CTA)
    try:
        B.dbw_select(h, dev(g.standard_exponential(n).astype(np.float32)), dev(np.full(n, 2, np.int32)))
        P, out = torch.zeros((n, n), device="cuda"), torch.full((n, ld), 3.0, device="cuda")
        B.dbw_get_weights(h, P)
        B.dbw_round(h, dev(x), out, 0.5, ext_grads=dev(gr))
        weights, xs, step = P.double().cpu().numpy(), x[:, :d].astype(np.float64), 0.5 * gr[:, :d].astype(np.float64)
        want = weights @ (xs - step) if order == "atc" else weights @ xs - step
        got = out.cpu().numpy()
    finally:
        B.dbw_destroy(h)
    # a weighted sum with weights that sum to one, and a step: a few rounding units of the largest terms
    np.testing.assert_allclose(got[:, :d], want, rtol=0, atol=16 * 2.0 ** -24 * np.abs(x).max())
    assert np.all(got[:, d:] == 3.0)
