"""GPU parity of the dense (matrix-core) mixing path against the CPU oracle, and its
agreement with the sparse path, through the C ABI."""
import numpy as np
import pytest
import torch

from paper_2102_06280_amd import inputs
from gpu_util import assert_params_close, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2102_06280_amd import binding
    return binding


def _graph(name):
    g = np.random.default_rng(211)
    return {"complete5": lambda: inputs.graph_complete(5), "complete40": lambda: inputs.graph_complete(40),
            "er100": lambda: inputs.graph_er(100, 0.6, g), "complete256": lambda: inputs.graph_complete(256),
            "complete130": lambda: inputs.graph_complete(130)}[name]()


CASES = [("complete5", 1000, 1024), ("complete40", 4100, 4160), ("er100", 2050, 2112),
         ("complete130", 777, 832), ("complete256", 8192 + 70, 8320), ("complete256", 64, 64),
         ("complete40", 30, 30)]


@pytest.mark.parametrize("order", [0, 1], ids=["cta", "atc"])
@pytest.mark.parametrize("gname,d,ld", CASES, ids=[f"{c[0]}-d{c[1]}" for c in CASES])
def test_dense_round_matches_oracle(B, orc, gname, d, ld, order):
    rowptr, colidx = _graph(gname)
    n = rowptr.size - 1
    deg = np.diff(rowptr)
    g = np.random.default_rng(213)
    h = B.dbw_create(rowptr, colidx, n, d, ld=ld, order=order, mix_path=B.MIX_DENSE)
    hs = B.dbw_create(rowptr, colidx, n, d, ld=ld, order=order, mix_path=B.MIX_CSR)
    try:
        assert B.dbw_mix_path(h) == B.MIX_DENSE and B.dbw_mix_path(hs) == B.MIX_CSR
        x = g.standard_normal((n, ld)).astype(np.float32)
        for rnd in range(3):
            gr = (g.standard_normal((n, ld)) * 0.01).astype(np.float32)
            t = g.standard_exponential(n).astype(np.float32)
            b = g.integers(0, deg // 2 + 1).astype(np.int32) if rnd else np.zeros(n, np.int32)
            lr = np.float32(0.05)
            dx, dg, dt, db = dev(x), dev(gr) if rnd < 2 else None, dev(t), dev(b)
            outs = []
            for hh in (h, hs):
                out = torch.full((n, ld), 7.0, dtype=torch.float32, device="cuda")
                B.dbw_select(hh, dt, db)
                B.dbw_round(hh, dx, out, lr, ext_grads=dg)
                outs.append(out.cpu().numpy())
            mask, p, _ = orc.select(rowptr, colidx, t, b)
            want = orc.round_(rowptr, colidx, mask, p, x, gr if rnd < 2 else None, lr, order, d=d)
            assert_params_close(outs[0], want, d=d, what=f"dense {gname} round {rnd}")
            assert_params_close(outs[1], want, d=d, what=f"sparse {gname} round {rnd}")
            assert np.all(outs[0][:, d:] == 7.0)
            x = want
            x[:, d:] = 0
    finally:
        B.dbw_destroy(h)
        B.dbw_destroy(hs)


def test_auto_path_choice(B):
    for graph, want in [(inputs.graph_complete(64), "dense"), (inputs.graph_ring(64), "csr")]:
        h = B.dbw_create(*graph, 64, 256)
        assert B.dbw_mix_path(h) == (B.MIX_DENSE if want == "dense" else B.MIX_CSR)
        B.dbw_destroy(h)
    rowptr, colidx = inputs.graph_ring(300)
    with pytest.raises(B.DbwError) as e:
        B.dbw_create(rowptr, colidx, 300, 64, mix_path=B.MIX_DENSE)
    assert e.value.code == B.ERR_UNSUPPORTED


def test_kernel_and_timing_name_of_every_size(B):
    """Rows on 16-byte boundaries: the fp32 instruction up to 32 workers, the split form above; off them: a thread per
    column up to 16, the split form above.  The names that the timing reports tell them apart."""
    for n, ld, want in [(16, 260, "mix_dense_kernel"), (32, 260, "mix_dense_kernel"), (33, 260, "mix_dense_split"),
                        (16, 257, "mix_dense_columns"), (17, 257, "mix_dense_split"), (33, 257, "mix_dense_split")]:
        h = B.dbw_create(*inputs.graph_complete(n), n, 257, ld=ld, mix_path=B.MIX_DENSE)
        try:
            x = torch.ones((n, ld), dtype=torch.float32, device="cuda")
            out = torch.zeros_like(x)
            B.dbw_select(h, dev(np.arange(n, dtype=np.float32)), dev(np.zeros(n, np.int32)))
            B.dbw_set_timing(h, True)
            B.dbw_round(h, x, out, 0.0)
            assert set(B.dbw_get_timing(h)) == {want}
            assert torch.allclose(out[:, :257], x[:, :257], rtol=0, atol=1e-5)
        finally:
            B.dbw_destroy(h)


# Worker counts at the edges of the four sizes of the kernel (32, 64, 128, 256 rows), columns at the edges of their
# tiles (256, 128, 64 and 32 columns) and of a float4, fewer and more tiles than compute units, rows with and without
# padding (the 4-byte loads).
EDGES = [(32, 255, 4), (33, 129, 1), (64, 128, 4), (65, 61, 4), (128, 64 * 257 + 3, 1), (129, 33, 1), (256, 32 * 256 + 31, 4),
         (256, 95, 1), (20, 517, 1), (200, 1, 4),
         # a thread per column or four of them: every size of its register block, a last group of one to three columns
         (2, 1, 1), (4, 1027, 1), (5, 257, 1), (16, 769, 1), (3, (1 << 19) - 1, 1), (8, (1 << 19) + 1, 1), (16, (1 << 19) + 3, 1),
         (9, (1 << 19) + 2, 1)]


@pytest.mark.parametrize("n,d,pad", EDGES, ids=[f"n{n}-d{d}-pad{p}" for n, d, p in EDGES])
def test_tile_edges_and_values_that_are_not_finite(B, orc, n, d, pad):
    """Both orders with a rate per worker against the oracle; then the same with an infinity and a NaN among the
    parameters: a row that waits for the infinite worker gets the infinity, every other row 0 * inf = NaN, and no
    other column changes.  Tolerance: the repository's 1e-5 per row, or where a row has so few columns that its sums
    can cancel, the first-order bound of an fp32 sum of n + 2 terms, (n + 2) 2^-24 times the sum of their magnitudes."""
    rowptr, colidx = inputs.graph_complete(n)
    deg = np.diff(rowptr)
    ld = (d + pad - 1) // pad * pad
    g = np.random.default_rng(1000 * n + d)
    x = g.standard_normal((n, ld)).astype(np.float32)
    gr = (g.standard_normal((n, ld)) * 0.01).astype(np.float32)
    eta = g.uniform(0.01, 0.1, n).astype(np.float32)
    t = g.standard_exponential(n).astype(np.float32)
    b = g.integers(0, deg // 2 + 1).astype(np.int32)
    mask, _, _ = orc.select(rowptr, colidx, t, b)
    bad = x.copy()
    j, c = n // 2, d // 2
    bad[j, c] = np.inf
    if d > 1:
        bad[n - 1, d - 1] = np.nan
    for order in (0, 1):
        h = B.dbw_create(rowptr, colidx, n, d, ld=ld, order=order, mix_path=B.MIX_DENSE)
        try:
            outs = []
            for v in (x, bad):
                out = torch.full((n, ld), 7.0, dtype=torch.float32, device="cuda")
                B.dbw_select(h, dev(t), dev(b))
                B.dbw_round_eta(h, dev(v), out, dev(eta), ext_grads=dev(gr))
                outs.append(out.cpu().numpy())
        finally:
            B.dbw_destroy(h)
        want = orc.round_eta(rowptr, colidx, mask, (deg - b).astype(np.int32), x, gr, eta, order, d=d)
        size = orc.round_(rowptr, colidx, mask, (deg - b).astype(np.int32), np.abs(x), None, 0.0, 0, d=d)
        bound = (n + 2) * 2.0 ** -24 * np.linalg.norm(size[:, :d], axis=1) / np.linalg.norm(want[:, :d], axis=1)
        assert_params_close(outs[0], want, d=d, tol=np.maximum(1e-5, bound), what=f"n {n} d {d} order {order}")
        assert np.all(outs[0][:, d:] == 7.0) and np.all(outs[1][:, d:] == 7.0)
        waits = np.array([i == j or bool(mask[rowptr[i] + (j if j < i else j - 1)]) for i in range(n)])
        assert np.all(outs[1][waits, c] == np.inf) and np.all(np.isnan(outs[1][~waits, c]))
        same = np.ones(ld, bool)
        same[c] = False
        if d > 1:
            same[d - 1] = False
            assert np.all(np.isnan(outs[1][:, d - 1]))
        assert np.array_equal(outs[0][:, same], outs[1][:, same])


@pytest.mark.parametrize("n,k", [(64, 1), (64, 2), (65, 1), (200, 1), (200, 2), (200, 5)])
def test_short_rows_are_as_exact_as_fp32_sums(B, n, k):
    """Rows of k + 1 terms (every worker waits for k neighbours): the root mean square of the error against 64 bits is at most that
    of fp32 multiply-adds in ascending order (5 % for the spread of the estimate over n x 20 000 sums)."""
    rowptr, colidx = inputs.graph_complete(n)
    d = 20_000
    g = np.random.default_rng(n + k)
    x = g.standard_normal((n, d)).astype(np.float32)
    h = B.dbw_create(rowptr, colidx, n, d, ld=d, mix_path=B.MIX_DENSE)
    try:
        out, P = torch.zeros((n, d), device="cuda"), torch.zeros((n, n), device="cuda")
        B.dbw_select(h, dev(g.permutation(n).astype(np.float32)), dev(np.full(n, n - 1 - k, np.int32)))
        B.dbw_round(h, dev(x), out, 0.0)
        B.dbw_get_weights(h, P)
        got, P = out.cpu().numpy(), P.cpu().numpy().astype(np.float64)
    finally:
        B.dbw_destroy(h)
    exact, size, plain = P @ x, P @ np.abs(x.astype(np.float64)), np.zeros((n, d), np.float32)
    assert np.all((P != 0).sum(1) == k + 1)
    for j in range(k + 1):
        at = np.array([np.flatnonzero(P[i])[j] for i in range(n)])
        plain = (plain + P[np.arange(n), at][:, None] * x[at].astype(np.float64)).astype(np.float32)
    rms = [np.sqrt(np.mean(((v - exact) / size) ** 2)) for v in (got, plain)]
    assert rms[0] <= 1.05 * rms[1], rms


def test_smallest_and_largest_values(B):
    """The largest float among the parameters stays finite, and values below 2^-110, of which the three bf16 values do not hold every
    bit, are off by at most 2^-133 each (next to the 2 x 2^-24 of a sum of two terms)."""
    n, d = 64, 1024
    rowptr, colidx = inputs.graph_complete(n)
    g = np.random.default_rng(9)
    x = (g.standard_normal((n, d)) * 2.0 ** -118).astype(np.float32)
    x[5, ::7] = np.finfo(np.float32).max
    x[9, 3::7] = -np.finfo(np.float32).max
    h = B.dbw_create(rowptr, colidx, n, d, ld=d, mix_path=B.MIX_DENSE)
    try:
        out, P = torch.zeros((n, d), device="cuda"), torch.zeros((n, n), device="cuda")
        B.dbw_select(h, dev(g.permutation(n).astype(np.float32)), dev(np.full(n, n - 2, np.int32)))
        B.dbw_round(h, dev(x), out, 0.0)
        B.dbw_get_weights(h, P)
        got, P = out.cpu().numpy().astype(np.float64), P.cpu().numpy().astype(np.float64)
    finally:
        B.dbw_destroy(h)
    assert np.isfinite(got).all()
    assert np.all(np.abs(got - P @ x) <= 2.0 ** -133 + 2.0 ** -23 * (P @ np.abs(x.astype(np.float64))))


@pytest.mark.parametrize("n,orders,pad", [(40, (0, 1, None), 64), (70, (0, None), 32), (100, (None,), 1), (200, (0, 1), 32),
                                          (200, (0,), 16)])
def test_matrices_around_the_last_level_cache(B, n, orders, pad):
    """Results (from 65 workers on: loads as well) pass the caches by once X, the result and the gradients together are larger than 256 MB and
    every row starts on a 128-byte line: the same bits in the columns that a matrix just below and one just above the line have in
    common, ragged ends and rows off the lines included."""
    rowptr, colidx = inputs.graph_complete(n)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    t, b = torch.rand(n, device="cuda", generator=gen), torch.full((n,), n // 3, dtype=torch.int32, device="cuda")
    for order in orders:                                # None: without gradients
        line = (256 << 20) // ((8 if order is None else 12) * n)
        sizes = [line - 999, line + 1003]
        x, gr = torch.empty(n, sizes[0], device="cuda").normal_(generator=gen), None
        if order is not None:
            gr = torch.empty(n, sizes[0], device="cuda").normal_(generator=gen)
        outs = []
        for d in sizes:
            ld = inputs.pad_ld(d, pad)
            assert ((8 if order is None else 12) * n * ld > 256 << 20) == (d == sizes[1])
            X, G = torch.zeros(n, ld, device="cuda"), None
            X[:, :sizes[0]] = x
            if gr is not None:
                G = torch.zeros(n, ld, device="cuda")
                G[:, :sizes[0]] = gr
            out = torch.full((n, ld), 7.0, device="cuda")
            h = B.dbw_create(rowptr, colidx, n, d, ld=ld, order=order or 0)
            try:
                assert B.dbw_mix_path(h) == B.MIX_DENSE
                B.dbw_select(h, t, b)
                B.dbw_round(h, X, out, 0.05, ext_grads=G)
                torch.cuda.synchronize()
            finally:
                B.dbw_destroy(h)
            assert bool((out[:, d:] == 7.0).all()) and bool((out[:, sizes[0]:d] == 0.0).all())
            outs.append(out[:, :sizes[0]])
        assert torch.equal(outs[0], outs[1])
        del outs, X, G, x, gr, out
