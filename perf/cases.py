"""The calls whose time matters, as a user's program makes them: one full-graph GNN layer on one GPU's share
(aggregation over a local and a halo table, then the dense Update), small whole models, the two halves of a
layer by themselves, and the embedding-bag sum of a recommendation batch.

Graphs are drawn on the GPU from the seed and handed to the library as host CSR arrays, the form
mgg_build_partition takes; a partition, weights, workspace and output buffers are kept by the caller, as a program
that runs a layer again and again (inference over all nodes, epochs, time steps) keeps them.
"""
import math

import numpy as np
import torch

from paper_2209_06800_amd import binding

DEV = "cuda"

# R-MAT corner probabilities: social-network-like skew, and the milder skew of a product graph
RMAT_SKEWED = (0.57, 0.19, 0.19, 0.05)
RMAT_MILD = (0.45, 0.22, 0.22, 0.11)


# ---- graphs ------------------------------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _canonical(n, s, t):
    """Undirected, no self-loops, no duplicates, sorted: host row_ptr (int64) and column (int32) arrays."""
    keep = s != t
    s, t = s[keep].long(), t[keep].long()
    key = torch.cat([s * n + t, t * n + s])
    del s, t
    key = torch.unique_consecutive(key.sort().values)
    row = torch.div(key, n, rounding_mode="floor")
    col = (key - row * n).int()
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.bincount(row, minlength=n).cumsum(0)
    return ptr.cpu().numpy(), col.cpu().numpy()


def _rmat(n, pairs, corners, g):
    scale = max(1, (n - 1).bit_length())
    a, b, c, _ = corners
    out, have = [], 0
    while have < pairs:
        k = int(min(1 << 24, (pairs - have) * (1.0 if n == 1 << scale else 1.4) + 1024))
        s = torch.zeros(k, dtype=torch.int32, device=DEV)
        t = torch.zeros(k, dtype=torch.int32, device=DEV)
        for _ in range(scale):
            r = torch.rand(k, device=DEV, generator=g)
            s = s * 2 + (r >= a + b)
            t = t * 2 + (((r >= a) & (r < a + b)) | (r >= a + b + c))
        ok = (s < n) & (t < n)
        s, t = s[ok][: pairs - have], t[ok][: pairs - have]
        out.append((s, t))
        have += s.numel()
    return torch.cat([p[0] for p in out]), torch.cat([p[1] for p in out])


def _power_law(n, d_min, d_max, g):
    """Chung-Lu pairs on expected degrees of a truncated power law (density exponent 2.1)."""
    u = torch.rand(n, dtype=torch.float64, device=DEV, generator=g)
    lo, hi = d_min ** -1.1, d_max ** -1.1
    w = (lo - u * (lo - hi)) ** (-1.0 / 1.1)
    cdf = w.cumsum(0)
    m = int(cdf[-1].item() / 2)
    cdf = cdf / cdf[-1]
    ends = []
    for _ in range(2):
        r = torch.rand(m, dtype=torch.float64, device=DEV, generator=g)
        ends.append(torch.searchsorted(cdf, r).clamp_(max=n - 1))
    return ends


def _uniform_pairs(n, pairs, g):
    return (torch.randint(0, n, (pairs,), device=DEV, generator=g), torch.randint(0, n, (pairs,), device=DEV, generator=g))


def _graph(case, g):
    n = case["nodes"]
    if case["graph"] == "power":
        s, t = _power_law(n, case["d_min"], case["d_max"], g)
    elif case["graph"] == "uniform":
        s, t = _uniform_pairs(n, case["pairs"], g)
    else:
        s, t = _rmat(n, case["pairs"], RMAT_SKEWED if case["graph"] == "rmat" else RMAT_MILD, g)
    return _canonical(n, s, t)


def _tables(case, rows, width, g, relu=False):
    """A table of embeddings ~ N(0, 1) (after a ReLU for the input of a second layer).  Rows lie end to end, as a
    plain contiguous tensor has them, or -- `padded` -- start on 128-byte boundaries."""
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    x = torch.randn(rows, width, device=DEV, generator=g)
    if relu:
        x.relu_()
    x = x.to(dt)
    if case.get("padded"):
        per = 128 // x.element_size()
        ld = -(-width // per) * per
        if ld != width:
            buf = torch.zeros(rows, ld, dtype=dt, device=DEV)
            buf[:, :width] = x
            x = buf[:, :width]
    return x


def _weight(case, d_in, d_out, g):
    w = torch.randn(d_in, d_out, device=DEV, generator=g) * 0.1
    return w.bfloat16() if case["dtype"] == "bf16" else w


# ---- the cases ---------------------------------------------------------------------------------------------
def listed():
    return [
        # One layer of a small graph (molecules, meshes, a sampled batch): latency and launches are all there is.
        dict(name="er4k_gcn16", kind="layer", graph="uniform", nodes=4096, pairs=32768, parts=1, mode="gcn", dtype="f32", d_in=16, d_hid=0, d_out=16,
             act="relu", order="agg_first"),
        # A whole 2-layer GCN with the softmax at its end, hidden width 16, on a citation-graph-sized input.
        dict(name="rmat30k_gcn2_softmax", kind="gcn2", graph="rmat_mild", nodes=30011, pairs=240000, parts=1, mode="gcn", dtype="f32", d_in=100, d_hid=16,
             d_out=7, act="relu", order="agg_first"),
        # One GPU's quarter of a skewed 2^20-node graph, GCN 64 -> 64.
        dict(name="rmat1M_gcn64_p4", kind="layer", graph="rmat", nodes=1 << 20, pairs=1 << 24, parts=4, mode="gcn", dtype="f32", d_in=64, d_hid=0, d_out=64,
             act="relu", order="agg_first"),
        # One GPU's eighth of a skewed 2^22-node graph in bf16, GIN with its MLP.
        dict(name="rmat4M_gin128_bf16_p8", kind="layer", graph="rmat", nodes=1 << 22, pairs=1 << 25, parts=8, mode="gin", dtype="bf16", d_in=128, d_hid=128,
             d_out=128, act="relu", order="agg_first"),
        # A dense power-law graph whole on one GPU, wide rows, aggregation first (the paper's order).
        dict(name="power233k_gcn602", kind="layer", graph="power", nodes=232965, d_min=115.5, d_max=20000.0, parts=1, mode="gcn", dtype="f32", d_in=602, d_hid=0,
             d_out=256, act="relu", order="agg_first", padded=True),
        # The same kind of layer when the caller lets the library choose the order; features as a plain contiguous tensor.
        dict(name="power120k_gcn602_auto", kind="layer", graph="power", nodes=120011, d_min=90.0, d_max=12000.0, parts=1, mode="gcn", dtype="f32", d_in=602,
             d_hid=0, d_out=256, act="relu", order="auto"),
        # The two layers of a GCN on one GPU's eighth of a product-graph-sized input: 100 -> 256 aggregated at 100 ...
        dict(name="rmat2.4M_gcn100_p8", kind="layer", graph="rmat_mild", nodes=2449029, pairs=61859140, parts=8, mode="gcn", dtype="f32", d_in=100, d_hid=0,
             d_out=256, act="relu", order="agg_first"),
        # ... and 256 -> 47 in the order the library chooses.
        dict(name="rmat2.4M_gcn256to47_p8", kind="layer", graph="rmat_mild", nodes=2449029, pairs=61859140, parts=8, mode="gcn", dtype="f32", d_in=256, d_hid=0,
             d_out=47, act="none", order="auto"),
        # Aggregation alone (a sum over neighbours feeding another library), an odd width in a plain contiguous tensor.
        dict(name="rmat260k_sum75", kind="aggregate", graph="rmat", nodes=260000, pairs=4000000, parts=2, mode="gin", dtype="f32", d_in=75, d_hid=0, d_out=75,
             act="none", order="agg_first"),
        # A recommendation batch: 26 tables, one lookup in each per sample, a quarter of the table on this GPU.
        dict(name="bags26_262k_dim64", kind="bags", tables=26, table_rows=1 << 18, samples=1 << 18, dtype="f32", d_in=64),
        # The dense half of a wide layer by itself, with bias.
        dict(name="update602to256_f32", kind="update", rows=232965, dtype="f32", d_in=602, d_hid=0, d_out=256, act="relu", padded=True),
        # GIN's MLP by itself on bf16 weights, fp32 rows in.
        dict(name="mlp128_bf16", kind="mlp", rows=524288, dtype="bf16", d_in=128, d_hid=128, d_out=128, act="relu"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo=8, hi=300):
    """Feature widths: half of them the round ones people choose, half whatever a data set has."""
    if rng.random() < 0.5:
        return rng.choice([w for w in (16, 32, 64, 96, 128, 192, 256) if lo <= w <= hi])
    return rng.randint(lo, hi)


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "gcn2", "aggregate", "bags", "update", "mlp"])
    if kind == "bags":
        return dict(kind="bags", tables=rng.randint(8, 40), table_rows=_log(rng, 1 << 12, 1 << 18), samples=_log(rng, 1 << 11, 1 << 18),
                    dtype=rng.choice(["f32", "bf16"]), d_in=rng.choice([16, 32, 64, 128, rng.randint(10, 120)]))
    if kind == "update":
        return dict(kind="update", rows=_log(rng, 2000, 400000), dtype=rng.choice(["f32", "f32", "bf16"]), d_in=_width(rng, 16, 602), d_hid=0,
                    d_out=_width(rng, 16, 256), act=rng.choice(["relu", "none"]), padded=rng.random() < 0.5)
    if kind == "mlp":
        return dict(kind="mlp", rows=_log(rng, 4000, 600000), dtype="bf16", d_in=rng.choice([64, 128, 128]), d_hid=rng.choice([64, 96, 128]),
                    d_out=rng.choice([40, 64, 128]), act="relu")
    nodes = _log(rng, 2000, 1500000)
    graph = rng.choice(["rmat", "rmat_mild", "power", "uniform"])
    c = dict(kind=kind, graph=graph, nodes=nodes)
    if graph == "power":
        c["nodes"] = nodes = min(nodes, 200000)
        c["d_min"] = float(_log(rng, 8, 90))
        c["d_max"] = float(max(4 * c["d_min"], nodes // 12))
    else:
        c["pairs"] = int(min(nodes * rng.uniform(6.0, 30.0), 24e6, nodes * (nodes - 1) / 8))
    c["parts"] = 1 if kind == "gcn2" else rng.choice([1, 1, 2, 4, 8])
    c["mode"] = "gcn" if kind == "gcn2" else rng.choice(["gcn", "gcn", "gin"])
    c["dtype"] = "f32" if kind == "gcn2" or c["mode"] == "gcn" and rng.random() < 0.75 else rng.choice(["f32", "bf16"])
    c["d_in"] = _width(rng)
    c["d_out"] = c["d_in"] if kind == "aggregate" else rng.randint(3, 64) if kind == "gcn2" else _width(rng, 16, 256)
    c["d_hid"] = rng.choice([16, 16, 64]) if kind == "gcn2" else _width(rng, 32, 128) if kind == "layer" and c["mode"] == "gin" else 0
    c["act"] = rng.choice(["relu", "none"]) if kind == "layer" else "relu" if kind == "gcn2" else "none"
    c["order"] = "auto" if kind != "aggregate" and rng.random() < 0.4 and c["dtype"] == "f32" else "agg_first"
    c["padded"] = rng.random() < 0.4
    return c


# ---- preparing and running ---------------------------------------------------------------------------------
def _layer_state(case, part, x_local, x_halo, weights, acts, g):
    s = dict(part=part, mode=case["mode"], x_local=x_local, x_halo=x_halo, weights=weights, acts=acts, order=case["order"], eps=0.1 if case["mode"] == "gin" else 0.0)
    need = binding.mgg_layer_workspace_bytes(part, case["mode"], weights, acts, eps=s["eps"], order=case["order"])
    s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    s["out"] = torch.empty(int(part.info.n_own), int(weights[-1].shape[1]), device=DEV)
    return s


def _prepare_bags(case, g):
    tables, rows, samples = case["tables"], case["table_rows"], case["samples"]
    # ranks by a truncated power law (exponent 1.05), then a shuffle of the rows of each table
    u = torch.rand(samples, tables, device=DEV, generator=g, dtype=torch.float64)
    e = 1 - 1.05
    rank = (((rows ** e - 1) * u + 1) ** (1 / e)).floor_().long().sub_(1).clamp_(0, rows - 1)
    perm = torch.stack([torch.randperm(rows, device=DEV, generator=g) for _ in range(tables)])
    idx = perm.t().gather(0, rank) + torch.arange(tables, device=DEV) * rows
    ptr = np.arange(0, (samples + 1) * tables, tables, dtype=np.int64)
    total = tables * rows
    part = binding.mgg_build_bags(ptr, idx.reshape(-1).int().cpu().numpy(), total, 0, total // 4)
    halo_rows = int(part.info.num_halo)
    s = dict(kind="bags", part=part, x_local=_tables(case, total // 4, case["d_in"], g), x_halo=_tables(case, halo_rows, case["d_in"], g) if halo_rows else None)
    s["out"] = torch.empty(samples, case["d_in"], device=DEV)
    return s


def prepare(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "bags":
        return _prepare_bags(case, g)
    if kind in ("update", "mlp"):
        dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        # the rows come out of an fp32 aggregation; bf16 belongs to the weights and the matrix product
        a = _tables(dict(case, dtype="f32"), case["rows"], case["d_in"], g)
        s = dict(kind=kind, a=a, act=case["act"], out=torch.empty(case["rows"], case["d_out"], device=DEV))
        s["bias"] = torch.randn(case["d_out"], device=DEV, generator=g) * 0.1
        if kind == "update":
            s["w"] = _weight(case, case["d_in"], case["d_out"], g)
        else:
            s["w1"] = _weight(case, case["d_in"], case["d_hid"], g)
            s["w2"] = _weight(case, case["d_hid"], case["d_out"], g)
            s["hidden"] = torch.empty(case["rows"], case["d_hid"], dtype=dt, device=DEV)
        return s
    row_ptr, col = _graph(case, g)
    part = binding.mgg_build_partition(row_ptr, col, case["parts"], 0)
    n_own, halo = int(part.info.n_own), int(part.info.num_halo)
    relu = case["d_in"] == 256                     # the input of a second layer
    x_local = _tables(case, n_own, case["d_in"], g, relu)
    x_halo = _tables(case, halo, case["d_in"], g, relu) if halo else None
    if kind == "aggregate":
        part.reserve(case["d_in"])
        return dict(kind=kind, part=part, mode=case["mode"], x_local=x_local, x_halo=x_halo, eps=0.1 if case["mode"] == "gin" else 0.0,
                    out=torch.empty(n_own, case["d_in"], device=DEV))
    if kind == "gcn2":
        w1, w2 = _weight(case, case["d_in"], case["d_hid"], g), _weight(case, case["d_hid"], case["d_out"], g)
        first = _layer_state(case, part, x_local, None, [w1], ["relu"], g)
        second = _layer_state(case, part, first["out"], None, [w2], ["softmax"], g)
        return dict(kind=kind, layers=[first, second])
    if case["d_hid"]:
        weights, acts = [_weight(case, case["d_in"], case["d_hid"], g), _weight(case, case["d_hid"], case["d_out"], g)], ["relu", case["act"]]
    else:
        weights, acts = [_weight(case, case["d_in"], case["d_out"], g)], [case["act"]]
    return dict(kind=kind, layers=[_layer_state(case, part, x_local, x_halo, weights, acts, g)])


def run(s):
    kind = s["kind"]
    if kind == "bags":
        return binding.mgg_bag_sum(s["part"], s["x_local"], s["x_halo"], out=s["out"])
    if kind == "update":
        return binding.mgg_update(s["a"], s["w"], s["bias"], s["act"], out=s["out"])
    if kind == "mlp":
        return binding.mgg_update_mlp(s["a"], s["w1"], s["w2"], (s["act"], "none"), (None, s["bias"]), hidden=s["hidden"], out=s["out"])
    if kind == "aggregate":
        return binding.mgg_aggregate(s["part"], s["mode"], s["x_local"], s["x_halo"], eps=s["eps"], out=s["out"])
    return [binding.mgg_layer_forward(l["part"], l["mode"], l["x_local"], l["x_halo"], l["weights"], l["acts"], eps=l["eps"], workspace=l["workspace"],
                                      out=l["out"], order=l["order"]) for l in s["layers"]]


# ---- what a pass cannot do without --------------------------------------------------------------------------
def _share(case):
    """About how many neighbours and halo rows the share of the case's graph has (duplicate pairs and the
    correlation of the two ends left out: right to some 15 %)."""
    n, p = case["nodes"], case["parts"]
    if case["graph"] == "power":
        lo, hi = case["d_min"], case["d_max"]
        mean = (lo ** -0.1 - hi ** -0.1) / 0.1 / ((lo ** -1.1 - hi ** -1.1) / 1.1)
        pairs, own = n * mean / 2, 1.0 / p
        touched = 1.0 - math.exp(-mean / p)
    elif case["graph"] == "uniform":
        pairs, own = case["pairs"], 1.0 / p
        touched = 1.0 - math.exp(-2.0 * pairs / n / p)
    else:
        a, b, c, d = RMAT_SKEWED if case["graph"] == "rmat" else RMAT_MILD
        pairs = case["pairs"]
        scale = max(1, (n - 1).bit_length())
        own = (a + b) ** math.log2(p * (1 << scale) / n) / (a + b) ** math.log2((1 << scale) / n)
        # nodes by the number of one bits in their id: how many of them some owned row gathers
        lam = [2.0 * pairs * own * (a + c) ** (scale - k) * (b + d) ** k for k in range(scale + 1)]
        touched = sum(math.comb(scale, k) * -math.expm1(-lam[k]) for k in range(scale + 1)) / (1 << scale)
    return 2.0 * pairs * own, n / p, (n - n / p) * touched


def work(case):
    kind, dt = case["kind"], 2 if case["dtype"] == "bf16" else 4
    d_in = case["d_in"]
    if kind == "bags":
        looks = case["tables"] * case["samples"]
        rows, e = case["table_rows"], 1 - 1.05
        # distinct rows: rank r of a table is drawn with density ~ r^-1.05
        edges = np.unique(np.round(np.logspace(0, math.log10(rows), 200)))
        mass = (edges[1:] ** e - edges[:-1] ** e) / (rows ** e - 1)
        width = edges[1:] - edges[:-1]
        distinct = case["tables"] * float(np.sum(width * -np.expm1(-case["samples"] * mass / width)))
        return {"bytes": distinct * d_in * dt + looks * 4 + case["samples"] * (d_in * 4 + 8), "flops": looks * d_in}
    if kind in ("update", "mlp"):
        widths = [d_in] + ([case["d_hid"]] if case["d_hid"] else []) + [case["d_out"]]
        macs = sum(x * y for x, y in zip(widths, widths[1:]))
        return {"bytes": case["rows"] * (d_in + case["d_out"]) * 4 + macs * dt, "flops": 2 * case["rows"] * macs}
    nnz, own, halo = _share(case)
    per_edge = 2 if case["mode"] == "gcn" else 1
    ids = nnz * (8 if case["mode"] == "gcn" else 4) + own * 12
    if kind == "aggregate":
        return {"bytes": (own + halo) * d_in * dt + ids + own * d_in * 4, "flops": nnz * d_in * per_edge}
    if kind == "gcn2":
        h, o = case["d_hid"], case["d_out"]
        return {"bytes": own * (d_in * 4 + h * 8 + o * 4) + 2 * ids, "flops": nnz * (min(d_in, h) + min(h, o)) * per_edge + 2 * own * (d_in * h + h * o)}
    widths = [d_in] + ([case["d_hid"]] if case["d_hid"] else []) + [case["d_out"]]
    macs = sum(x * y for x, y in zip(widths, widths[1:]))
    gathered = min(widths[:2]) if case["order"] == "auto" else d_in
    return {"bytes": (own + halo) * d_in * dt + ids + own * case["d_out"] * 4 + macs * dt, "flops": nnz * gathered * per_edge + 2 * own * macs}


def tolerance(case):
    """About four times the distance to the same path evaluated in float64 (2-norms): 1.7e-3 to 2.4e-3 with one bf16
    rounding per matrix operand, 0.9e-7 to 4.7e-7 where sums and products are fp32 (the most at 602 terms)."""
    if case["dtype"] == "bf16" and case["kind"] != "aggregate" and case["kind"] != "bags":
        return {"rel": 1e-2}
    return {"rel": 2e-6}
