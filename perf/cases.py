"""Performance cases of the training round: what a program that simulates N workers asks of the library.

Every case is one call sequence through the public entry points of paper_2102_06280_amd.binding on inputs that
already live on the GPU.  Three kinds:

  round  dbw_select, then dbw_round (or dbw_round_eta): one training round of all workers, with the model's own
         gradients or with gradients supplied by the caller
  tail   dbw_consensus_rounds: several gradient-free rounds at once (the consensus-only iterations after training)
  run    a short training run from the first round on: the threshold rule chooses the backup counts of every round
         after the first, the round's duration is recorded

A case is a dict of plain values; listed() holds the ones that are looked at by name, draw() makes others of the
same ranges.  prepare() makes the inputs and the context, run() is one pass, exact() the same results in 64 bits.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2102_06280_amd import binding as B
from paper_2102_06280_amd import inputs

# --------------------------------------------------------------------------- the cases

_BASE = {"kind": "round", "workers": 8, "graph": "ring", "degree": 0.0, "backup": 1, "times": "exp", "model": "none",
         "dims": "", "batch": 0, "loss": "xent", "d": 0, "pad": 64, "order": "cta", "layout": "rows",
         "rates": "one", "gradients": True, "rounds": 1, "lr": 0.05}


def _case(name=None, **kw):
    assert set(kw) <= set(_BASE), kw
    c = {**_BASE, **kw}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest training round: logistic regression on 784 inputs, eight workers on a ring.  A simulation runs
        # thousands of these; launches and their latency are all there is.
        _case("softmax-ring8", model="mlp", dims="784,10", batch=32),
        # A whole short training run of the logistic regression on 256 inputs with the threshold rule: 20 rounds,
        # each with its own response times and batch, and the durations that the loss is plotted against.
        _case("lrm6-threshold-run20", kind="run", workers=6, graph="er", degree=0.5, times="lognormal", model="mlp",
              dims="256,10", batch=1024, lr=0.2, rounds=20),
        # A one-hidden-layer perceptron on a short batch, 32 workers.
        _case("mlp-reg32-short-batch", workers=32, graph="regular", degree=4, backup=2, times="shifted", model="mlp",
              dims="784,200,10", batch=64),
        # The two-hidden-layer network on a long batch, squared error, local step first.
        _case("2nn-er10-long-batch", workers=10, graph="er", degree=0.4, backup=2, times="lognormal", model="mlp",
              dims="256,256,256,10", batch=1024, loss="mse", order="atc", lr=1.0),
        # A perceptron whose widths, batch, class count and row length divide by nothing, on rows without padding
        # (the default row stride), a learning rate per worker.
        _case("mlp-er20-odd-widths", workers=20, graph="er", degree=0.25, backup=3, model="mlp",
              dims="617,301,75,26", batch=101, pad=1, rates="each"),
        # The convolutional network on 3 x 32 x 32 images, 64 workers.
        _case("cnn-er64-colour", workers=64, graph="er", degree=0.1, backup=3, times="lognormal", model="cnn",
              dims="3,32,32,32,64,5,512,10", batch=32, lr=0.01),
        # The same kind of network on 1 x 28 x 28 images with other widths: no shape that anything is specialised on.
        _case("cnn-reg16-grey", workers=16, graph="regular", degree=4, backup=2, model="cnn",
              dims="1,28,28,16,32,5,128,10", batch=50, lr=0.01),
        # Averaging and step alone on an 11.2 M parameter vector per worker, gradients supplied, tile-major storage.
        _case("consensus-reg128-tiles", workers=128, graph="regular", degree=8, backup=4, d=11_200_000, layout="tiles"),
        # The same on plain rows, local step first.
        _case("consensus-reg128-rows", workers=128, graph="regular", degree=8, backup=4, d=2_800_000, order="atc"),
        # Plain rows of odd length without padding: what a caller gets who passes d and nothing else.
        _case("consensus-er48-odd-rows", workers=48, graph="er", degree=0.15, backup=3, d=1_000_003, pad=1),
        # Complete graph, up to half of the neighbours left out as backups: the matrix form of the averaging.
        _case("consensus-complete256", workers=256, graph="complete", backup=128, d=1_000_000),
        # Eight gradient-free rounds after the training phase, applied in one pass.
        _case("tail8-reg128", kind="tail", workers=128, graph="regular", degree=8, backup=4, d=2_800_000,
              gradients=False, rounds=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, n):
    kind = rng.choice(["ring", "regular", "er", "complete"]) if n <= 256 else "regular"
    if n < 6 or kind == "ring":
        return {"graph": "ring" if n > 2 else "complete", "degree": 0.0, "backup": rng.randint(0, 1)}
    if kind == "complete":
        return {"graph": "complete", "degree": 0.0, "backup": n // 2}
    if kind == "regular":
        k = rng.choice([k for k in (3, 4, 6, 8) if k < n - 1 and n * k % 2 == 0])
        return {"graph": "regular", "degree": k, "backup": k // 2}
    # dense enough to be connected after a few attempts
    p = round(min(0.9, rng.uniform(1.5, 3.0) * math.log(n) / n + 0.05), 3)
    return {"graph": "er", "degree": p, "backup": max(1, int(p * n / 3))}


_COST_CAP = 1.5e9          # worker x parameter products of the averaging kinds (the largest listed: 1.43e9)
_FLOP_CAP = 2.0e11         # gradient operations (the largest listed: 2.07e11)


def draw(rng: random.Random):
    """One more case: any kind, sizes spread over their logarithm between the smallest and largest listed ones."""
    while True:
        family = rng.choice(["mix", "mix", "tail", "mlp", "mlp", "cnn", "run"])
        order = rng.choice(["cta", "atc"])
        times = rng.choice(["exp", "shifted", "lognormal"])
        if family in ("mix", "tail"):
            n = _log_int(rng, 4, 256)
            d = _log_int(rng, 5_000, 11_200_000)
            pad = rng.choice([64, 64, 64, 1])
            layout = "tiles" if family == "mix" and pad == 64 and rng.random() < 0.4 else "rows"
            c = _case(kind="tail" if family == "tail" else "round", workers=n, d=d, pad=pad, layout=layout, order=order,
                      times=times, rates=rng.choice(["one", "one", "each"]) if family == "mix" else "one",
                      gradients=family == "mix" and rng.random() < 0.85,
                      rounds=rng.randint(2, 12) if family == "tail" else 1, **_draw_graph(rng, n))
            if not c["gradients"]:
                c["rates"] = "one"
            if n * d <= _COST_CAP:
                return c
        elif family in ("mlp", "run"):
            n = _log_int(rng, 4, 64) if family == "mlp" else _log_int(rng, 4, 24)
            depth = rng.choice([0, 1, 1, 2, 2, 3])
            width = _log_int(rng, 32, 512)
            equal = rng.random() < 0.5
            hidden = [width if equal else _log_int(rng, 32, 512) for _ in range(depth)]
            if rng.random() < 0.6:                   # most networks have widths of a round number
                hidden = [max(32, 64 * round(h / 64)) for h in hidden] if rng.random() < 0.5 else \
                         [max(32, 4 * round(h / 4)) for h in hidden]
            first = rng.choice([256, 784, _log_int(rng, 32, 1024)])
            classes = rng.choice([10, 10, rng.randint(2, 40)])
            batch = rng.choice([32, 64, 256, 1024, _log_int(rng, 8, 1024)])
            if family == "run":
                hidden, batch = [], min(batch, 1024)
            c = _case(kind="run" if family == "run" else "round", workers=n, model="mlp",
                      dims=",".join(map(str, [first] + hidden + [classes])), batch=batch,
                      loss=rng.choice(["xent", "xent", "mse"]), pad=rng.choice([64, 64, 1]), order=order, times=times,
                      rates="one" if family == "run" else rng.choice(["one", "one", "each"]),
                      rounds=rng.randint(8, 20) if family == "run" else 1, **_draw_graph(rng, n))
            if work(c)["flops"] <= _FLOP_CAP:
                return c
        else:
            n = _log_int(rng, 4, 64)
            grey = rng.random() < 0.5
            size = rng.choice([16, 20, 24, 28, 32])
            c1, c2 = rng.choice([8, 12, 16, 32]), rng.choice([16, 24, 32, 64])
            dims = [1 if grey else 3, size, size, c1, c2, rng.choice([3, 5, 5]), _log_int(rng, 48, 512), 10]
            if rng.random() < 0.3:
                dims = [3, 32, 32, 32, 64, 5, 512, 10]
            c = _case(workers=n, model="cnn", dims=",".join(map(str, dims)), batch=rng.choice([16, 32, 32, _log_int(rng, 8, 64)]),
                      pad=rng.choice([64, 64, 1]), order=order, times=times, lr=0.01, **_draw_graph(rng, n))
            if work(c)["flops"] <= _FLOP_CAP:
                return c


# --------------------------------------------------------------------------- sizes


def _dims(case):
    return [int(v) for v in case["dims"].split(",")] if case["dims"] else []


def _desc(case):
    """The model as inputs.py describes it (None without a model)."""
    v = _dims(case)
    if case["model"] == "mlp":
        return {"kind": "mlp", "dims": v, "loss": case["loss"]}
    if case["model"] == "cnn":
        return {"kind": "cnn", "in": tuple(v[:3]), "c1": v[3], "c2": v[4], "k": v[5], "fc": v[6], "classes": v[7]}
    return None


def _sizes(case):
    desc = _desc(case)
    d = inputs.param_count(desc) if desc else case["d"]
    return d, inputs.pad_ld(d, case["pad"]), desc


def _graph(case, g):
    n, kind = case["workers"], case["graph"]
    if kind == "ring":
        return inputs.graph_ring(n)
    if kind == "complete":
        return inputs.graph_complete(n)
    if kind == "regular":
        return inputs.graph_regular(n, int(case["degree"]), g)
    return inputs.graph_er(n, float(case["degree"]), g)


def _mean_degree(case):
    n = case["workers"]
    return {"ring": 2.0, "complete": n - 1.0, "regular": float(case["degree"]), "er": case["degree"] * (n - 1)}[case["graph"]]


def _gradient_work(case):
    """(floats read and written, operations) of all workers' gradients: the products of the forward pass, of the weight
    gradients and of the data gradients that a layer above the first one needs."""
    n, batch, v = case["workers"], case["batch"], _dims(case)
    if case["model"] == "mlp":
        prod = [a * b for a, b in zip(v[:-1], v[1:])]
        return n * batch * (v[0] + 1), 2.0 * n * batch * (3 * sum(prod) - prod[0])
    c0, h, w, c1, c2, k, f, nc = v
    conv1 = h * w * c1 * c0 * k * k
    conv2 = (h // 2) * (w // 2) * c2 * c1 * k * k
    fc = c2 * (h // 4) * (w // 4) * f + f * nc
    return n * batch * (c0 * h * w + 1), 2.0 * n * batch * (2 * conv1 + 3 * conv2 + 3 * fc)


def work(case):
    n = case["workers"]
    d, _, _ = _sizes(case)
    selected = max(0.0, _mean_degree(case) - case["backup"] / 2.0)
    mix = 2.0 * n * d * (selected + 1 + (1 if case["gradients"] else 0))
    if case["kind"] == "tail":                      # one product of the rounds' matrices, or the rounds one by one
        return {"bytes": 8.0 * n * d, "flops": min(case["rounds"] * mix, 2.0 * n * n * d)}
    floats, flops = (2.0 + (1 if case["gradients"] and case["model"] == "none" else 0)) * n * d, mix
    if case["model"] != "none":
        f, o = _gradient_work(case)
        floats, flops = floats + f, flops + o
    return {"bytes": 4.0 * floats * case["rounds"], "flops": flops * case["rounds"]}


def tolerance(case):
    """Against results of fp32 arithmetic in another order of the sums."""
    if case["model"] == "none":
        # one weighted sum per value: a few rounding units of 6e-8
        return {"rel": 1e-6, "max": 2e-5}
    # The parameters after a round carry the rounding of the gradients times the learning rate (6e-8 of the result), and a
    # ReLU input or a pair of pooled values within rounding of a tie may fall to the other side in single samples: against
    # 64 bits up to 2.5e-6 was seen for the perceptrons (one unit of one sample) and 2e-6 to 1.3e-5, largest element 6e-3,
    # for the convolutional network, where some of its 25 million such decisions turn in every round.
    if case["model"] == "cnn":
        return {"rel": 5e-5, "max": 3e-2}
    return {"rel": 1e-5, "max": 5e-3}


# --------------------------------------------------------------------------- inputs


class _Context:
    """A context of the library, released with the state that holds it."""

    def __init__(self, *args, **kw):
        self.h = B.dbw_create(*args, **kw)

    def __del__(self):
        h, self.h = getattr(self, "h", None), None
        if h is not None:
            B.dbw_destroy(h)


def _rng(seed, what):
    return np.random.Generator(np.random.Philox(key=[int(seed) & 0xFFFFFFFFFFFFFFFF, what]))


def _response_times(case, g):
    n, r = case["workers"], case["rounds"]
    if case["times"] == "exp":
        t = g.standard_exponential((r, n))
    elif case["times"] == "shifted":
        t = 0.5 + g.standard_exponential((r, n))
    else:                                           # a tenth of the workers, at least one, five times slower throughout
        t = g.lognormal(0.0, 0.5, (r, n))
        t[:, g.choice(n, size=max(1, n // 10), replace=False)] *= 5.0
    return t.astype(np.float32)


def _host_inputs(case, seed):
    """Graph, response times, backup counts and learning rates."""
    rowptr, colidx = _graph(case, _rng(seed, 1))
    t = _response_times(case, _rng(seed, 2))
    deg = np.diff(rowptr)
    b = np.minimum(_rng(seed, 3).integers(0, case["backup"] + 1, (case["rounds"], case["workers"])), deg[None, :])
    if case["kind"] == "run":
        b = np.zeros_like(b)                        # every worker waits for all in round 1; the rule fills the others
    eta = (case["lr"] * _rng(seed, 4).uniform(0.5, 1.5, case["workers"])).astype(np.float32)
    return rowptr, colidx, t, b.astype(np.int32), eta


def _device_inputs(case, seed, device):
    """Parameters [N, ld] with zero padding, and the gradients or batches that go with them (rows layout)."""
    n, r = case["workers"], case["rounds"]
    d, ld, desc = _sizes(case)
    gen = torch.Generator(device=device)
    gen.manual_seed(int(seed) % (1 << 62))
    x = torch.zeros((n, ld), dtype=torch.float32, device=device)
    if desc is None:
        x[:, :d].normal_(0.0, 1.0, generator=gen)
        grads = None
        if case["gradients"]:
            grads = torch.zeros_like(x)
            grads[:, :d].normal_(0.0, 0.01, generator=gen)
        return x, grads, None, None
    off = 0
    for fan_in, nw, nb in inputs.layer_shapes(desc):
        x[:, off:off + nw].normal_(0.0, math.sqrt(2.0 / fan_in), generator=gen)
        x[:, off + nw:off + nw + nb].normal_(0.0, 0.1, generator=gen)
        off += nw + nb
    in_dim = desc["dims"][0] if desc["kind"] == "mlp" else int(np.prod(desc["in"]))
    classes = desc["dims"][-1] if desc["kind"] == "mlp" else desc["classes"]
    bx = torch.empty((r, n, case["batch"], in_dim), dtype=torch.float32, device=device).normal_(0.0, 1.0, generator=gen)
    by = torch.randint(0, classes, (r, n, case["batch"]), dtype=torch.int32, device=device, generator=gen)
    return x, None, bx, by


def prepare(case, seed):
    device = torch.device("cuda")
    n = case["workers"]
    d, ld, desc = _sizes(case)
    rowptr, colidx, t, b, eta = _host_inputs(case, seed)
    model = None
    if case["model"] == "mlp":
        model = B.make_model(B.MODEL_MLP, case["batch"], desc["dims"], B.LOSS_MSE if case["loss"] == "mse" else B.LOSS_XENT)
    elif case["model"] == "cnn":
        model = B.make_model(B.MODEL_CNN, case["batch"], _dims(case))
    layout = B.LAYOUT_TILES if case["layout"] == "tiles" else B.LAYOUT_ROWS
    ctx = _Context(rowptr, colidx, n, d, ld=ld, order=B.ORDER_ATC if case["order"] == "atc" else B.ORDER_CTA, model=model,
                   layout=layout)
    x, grads, bx, by = _device_inputs(case, seed, device)
    if layout == B.LAYOUT_TILES:
        for k, a in enumerate((x, grads)):
            if a is None:
                continue
            tiles = torch.empty_like(a)
            B.dbw_convert_layout(ctx.h, a, tiles, True)
            if k == 0:
                x = tiles
            else:
                grads = tiles
    s = {"case": case, "ctx": ctx, "x": x, "out": torch.zeros_like(x), "grads": grads, "bx": bx, "by": by,
         "t": torch.from_numpy(t).to(device), "b": torch.from_numpy(b).to(device),
         "eta": torch.from_numpy(eta).to(device) if case["rates"] == "each" else None}
    if case["model"] != "none":
        s["loss"] = torch.zeros((case["rounds"], n), dtype=torch.float32, device=device)
    if case["kind"] == "run":
        s["work"] = torch.zeros_like(x)
        s["duration"] = torch.zeros((case["rounds"], 2), dtype=torch.float32, device=device)
    return s


# --------------------------------------------------------------------------- one pass


def run(s):
    case, h = s["case"], s["ctx"].h
    if case["kind"] == "tail":
        B.dbw_consensus_rounds(h, s["x"], s["out"], s["t"], s["b"], case["rounds"])
        return s["out"]
    if case["kind"] == "run":
        B.dbw_dtur_reset(h)
        src, rest = s["x"], [s["out"], s["work"]]
        for r in range(case["rounds"]):
            if r == 0:
                B.dbw_select(h, s["t"][r], s["b"][r])
            else:
                B.dbw_dtur_select(h, s["t"][r], s["b"][r])
            dst = rest[r % 2]
            B.dbw_round(h, src, dst, _rate(case, r), batch_x=s["bx"][r], batch_y=s["by"][r], loss_out=s["loss"][r])
            B.dbw_round_time(h, s["duration"][r])
            src = dst
        return {"params": src, "loss": s["loss"], "backup": s["b"], "duration": s["duration"]}
    B.dbw_select(h, s["t"][0], s["b"][0])
    if case["model"] == "none":
        if s["eta"] is not None:
            B.dbw_round_eta(h, s["x"], s["out"], s["eta"], ext_grads=s["grads"])
        else:
            B.dbw_round(h, s["x"], s["out"], case["lr"], ext_grads=s["grads"])
        return s["out"]
    if s["eta"] is not None:
        B.dbw_round_eta(h, s["x"], s["out"], s["eta"], batch_x=s["bx"][0], batch_y=s["by"][0], loss_out=s["loss"][0])
    else:
        B.dbw_round(h, s["x"], s["out"], case["lr"], batch_x=s["bx"][0], batch_y=s["by"][0], loss_out=s["loss"][0])
    return {"params": s["out"], "loss": s["loss"]}


def _rate(case, r):
    """Learning rate of round r of a run: decayed by 0.95 per round."""
    return case["lr"] * 0.95 ** r


# --------------------------------------------------------------------------- the same in 64 bits


def _select(rowptr, colidx, t, b):
    """Selected neighbours of every worker, and the weight matrix in 64 bits."""
    n = rowptr.size - 1
    chosen = []
    for i in range(n):
        nb = colidx[rowptr[i]:rowptr[i + 1]]
        p = nb.size - int(b[i])
        chosen.append(np.sort(nb[np.lexsort((nb, t[nb]))][:p]))
    P = np.zeros((n, n))
    for i in range(n):
        for j in chosen[i]:
            P[i, j] = 1.0 / (1 + max(chosen[i].size, chosen[j].size))
        P[i, i] = 1.0 - P[i].sum()
    return chosen, P


def _tree_links(rowptr, colidx):
    """Breadth-first spanning tree from worker 0, neighbours ascending, links in the order of discovery."""
    seen, queue, links = {0}, [0], []
    for u in queue:
        for v in colidx[rowptr[u]:rowptr[u + 1]]:
            if int(v) not in seen:
                seen.add(int(v))
                queue.append(int(v))
                links.append((u, int(v)))
    return links


def _threshold_rule(rowptr, colidx, links, visited, t):
    """Backup counts of one round; `visited` (a set of link numbers) is updated."""
    if len(visited) == len(links):
        visited.clear()
    _, e = min((max(t[u], t[v]), e) for e, (u, v) in enumerate(links) if e not in visited)
    theta = max(t[links[e][0]], t[links[e][1]])
    visited.add(e)
    n = rowptr.size - 1
    b = np.zeros(n, dtype=np.int32)
    for j in range(n):
        nb = colidx[rowptr[j]:rowptr[j + 1]]
        b[j] = nb.size - (int((t[nb] <= theta).sum()) if t[j] <= theta else 0)
    return b


def _gradients(case, desc, x, bx, by):
    """(gradients [N, ld], mean losses [N]) by autograd in float64, one worker after the other."""
    d, _, _ = _sizes(case)
    grads, losses = torch.zeros_like(x), []
    for i in range(case["workers"]):
        theta = x[i, :d].clone().requires_grad_(True)
        off, layers = 0, []
        for fan_in, nw, nb in inputs.layer_shapes(desc):
            layers.append((theta[off:off + nw].view(nb, fan_in), theta[off + nw:off + nw + nb]))
            off += nw + nb
        a = bx[i].double()
        if desc["kind"] == "cnn":
            a = a.view(-1, *desc["in"])
            k = desc["k"]
            for wt, bias in layers[:2]:
                _, _, h, w = a.shape
                cols = torch.nn.functional.unfold(a, k, padding=k // 2)                # [batch, C k k, h w]
                cols = cols.transpose(1, 2).reshape(-1, wt.shape[1])
                z = (cols @ wt.t() + bias).view(-1, h * w, wt.shape[0]).transpose(1, 2)
                a = torch.nn.functional.max_pool2d(torch.relu(z.reshape(-1, wt.shape[0], h, w)), 2)
            a, layers = a.flatten(1), layers[2:]
        for l, (wt, bias) in enumerate(layers):
            a = a @ wt.t() + bias
            if l + 1 < len(layers):
                a = torch.relu(a)
        y = by[i].long()
        if case["loss"] == "mse":
            one = torch.nn.functional.one_hot(y, a.shape[1]).double()
            loss = (torch.softmax(a, 1) - one).square().sum(1).mean()
        else:
            loss = torch.nn.functional.cross_entropy(a, y)
        grads[i, :d] = torch.autograd.grad(loss, theta)[0]
        losses.append(loss.detach())
    return grads, torch.stack(losses)


def _average(P, x, d, step=None, order="cta"):
    """P (x - step) or P x - step over columns [0, d), a block of columns at a time; zero elsewhere."""
    out = torch.zeros(x.shape, dtype=torch.float64, device=x.device)
    width = max(1, (1 << 27) // x.shape[0])
    for lo in range(0, d, width):
        hi = min(d, lo + width)
        v = x[:, lo:hi].double()
        s = step(lo, hi) if step is not None else None
        if s is not None and order == "atc":
            v = v - s
        v = P @ v
        out[:, lo:hi] = v - s if s is not None and order == "cta" else v
    return out


def exact(case, seed):
    device = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    n = case["workers"]
    d, ld, desc = _sizes(case)
    rowptr, colidx, t, b, eta = _host_inputs(case, seed)
    x, grads, bx, by = _device_inputs(case, seed, device)

    def rate(r):
        if case["rates"] == "each":
            return torch.from_numpy(eta).double().to(device)[:, None]
        lr = _rate(case, r) if case["kind"] == "run" else case["lr"]
        return torch.full((n, 1), float(np.float32(lr)), dtype=torch.float64, device=device)

    def weights(r, bk):
        return torch.from_numpy(_select(rowptr, colidx, t[r], bk)[1]).to(device)

    if case["kind"] == "tail":
        P = torch.eye(n, dtype=torch.float64, device=device)
        for r in range(case["rounds"]):
            P = weights(r, b[r]) @ P
        return _average(P, x, d)
    if case["kind"] == "run":
        links, visited = _tree_links(rowptr, colidx), set()
        losses, counts, durations = [], [], []
        x = x.double()
        for r in range(case["rounds"]):
            bk = b[r] if r == 0 else _threshold_rule(rowptr, colidx, links, visited, t[r])
            g, loss = _gradients(case, desc, x, bx[r], by[r])
            step = rate(r) * g
            x = _average(weights(r, bk), x, d, lambda lo, hi: step[:, lo:hi], case["order"])
            chosen, _ = _select(rowptr, colidx, t[r], bk)
            wait = np.array([max([t[r][i]] + [t[r][j] for j in chosen[i]]) for i in range(n)])
            listed_ = sorted({int(j) for s in chosen for j in s})
            durations.append([wait.max(), max([wait[j] for j in listed_], default=0.0)])
            losses.append(loss)
            counts.append(bk)
        return {"params": x, "loss": torch.stack(losses), "backup": torch.from_numpy(np.stack(counts).astype(np.int32)),
                "duration": torch.tensor(np.array(durations, dtype=np.float64))}
    if desc is None:
        step = (lambda lo, hi: rate(0) * grads[:, lo:hi].double()) if grads is not None else None
        out = _average(weights(0, b[0]), x, d, step, case["order"])
        if case["layout"] == "tiles":
            w = B.TILE_COLUMNS
            out = out.view(n, ld // w, w).transpose(0, 1).contiguous().view(n, ld)
        return out
    x = x.double()
    g, loss = _gradients(case, desc, x, bx[0], by[0])
    step = rate(0) * g
    out = _average(weights(0, b[0]), x, d, lambda lo, hi: step[:, lo:hi], case["order"])
    return {"params": out, "loss": loss[None]}
