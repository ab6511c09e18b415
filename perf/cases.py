"""The calls that users of the library make, as cases to be timed and compared.

Each case is a plain dict.  `kind` names what the program does:

  spmm     aggregation Y = act(A X) on a plan that is kept (inference, serving)
  layer    one GCN layer act(A (X W)) on a kept plan
  build    a new matrix: partition it, then one aggregation (the benchmark's step)
  forward  a two-layer GCN forward on a kept plan (update, fused junction, aggregation)
  train    one training step on a kept plan: forward, loss, backward, both weight gradients
  values   the values of an aggregation matrix on a structure
  reload   a plan saved to bytes and loaded again on the same structure, then one aggregation

`graph` is "rmat" (power-law, shuffled ids; n nodes, m undirected edges, every node with its
self-loop) or "sbm" (dense communities of contiguous ids with power-law bridges).  Graphs are
made on the GPU from the seed; values are the symmetric GCN normalisation.
"""
import math

import numpy as np
import torch

import paper_2609_01983_amd as dg

DEV = "cuda:0"


def listed():
    return [
        # the smallest workload of the configurations: one aggregation of a graph of a few
        # thousand nodes, where the launch and the longest row are all there is
        dict(name="spmm_tiny", kind="spmm", graph="rmat", n=4096, m=32768, F=16, relu=False, bf16=False),
        # a layer of a small graph (ragged n) in inference: fp32 features in, bfloat16 out
        dict(name="layer_small", kind="layer", graph="rmat", n=20001, m=90000, F=256, F2=64, relu=True,
             xbf16=False, bf16=True),
        # the second workload: partition and one aggregation, n = 2^17, average degree 10
        dict(name="build_small", kind="build", graph="rmat", n=1 << 17, m=(1 << 17) * 9 // 2, F=64,
             walks=16, steps=5),
        # the paper's walk parameters (50 walks of 30 steps) on a graph of the paper's smallest
        # size (50K nodes, 1.2M entries), features of 96
        dict(name="build_paper_walks", kind="build", graph="rmat", n=50001, m=575000, F=96,
             walks=50, steps=30),
        # the third workload: a block-structured graph with local ids, F = 128
        dict(name="spmm_sbm", kind="spmm", graph="sbm", n=1 << 18, m=1 << 18, F=128, relu=False, bf16=False),
        # an output layer's aggregation: as many features as classes, an odd number, ragged n
        dict(name="spmm_odd", kind="spmm", graph="rmat", n=200003, m=1600000, F=47, relu=False, bf16=False),
        # training of a small graph, fp32 features: launches and small products
        dict(name="train_small", kind="train", graph="rmat", n=30007, m=210000, F=128, F2=64, F3=32,
             xbf16=False),
        # training at the flagship's widths on a graph of half a million nodes, bfloat16 features
        dict(name="train_medium", kind="train", graph="rmat", n=1 << 19, m=(1 << 19) * 15 // 2, F=256,
             F2=128, F3=64, xbf16=True),
        # another aggregator on a large structure (its values are filled before a plan is built)
        dict(name="values_gcn", kind="values", graph="rmat", n=1 << 20, m=(1 << 20) * 29 // 2, agg="gcn"),
        # a job that resumes: the plan saved by the last run is loaded and used
        dict(name="reload_medium", kind="reload", graph="rmat", n=1 << 20, m=(1 << 20) * 15 // 2, F=64,
             walks=16, steps=5),
        # the fourth workload: partition and one aggregation, n = 2^21, average degree 30
        dict(name="build_large", kind="build", graph="rmat", n=1 << 21, m=(1 << 21) * 29 // 2, F=128,
             walks=16, steps=5),
        # the flagship workload's forward on its kept plan: 256 -> 128 -> 64, n = 2^22
        dict(name="forward_large", kind="forward", graph="rmat", n=1 << 22, m=(1 << 22) * 15 // 2,
             F=256, F2=128, F3=64, xbf16=False),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["spmm", "spmm", "layer", "build", "build", "forward", "train", "values", "reload"])
    graph = "sbm" if rng.random() < 0.2 else "rmat"
    n = log_int(1 << 12, 1 << 18 if graph == "sbm" else 1 << 21)
    m = n if graph == "sbm" else int(n * rng.uniform(1.5, 14.5))
    c = dict(kind=kind, graph=graph, n=n, m=m)
    widths = [32, 64, 96, 128, 160, 256]
    if kind in ("spmm", "build", "reload"):
        c["F"] = rng.choice([16, 32, 64, 100, 128, rng.randint(3, 128), rng.randint(3, 128)])
    if kind == "spmm":
        c.update(relu=rng.random() < 0.5, bf16=rng.random() < 0.5)
    if kind in ("build", "reload"):
        c.update(walks=rng.choice([8, 16, 50]), steps=rng.choice([4, 5, 5, 12]))
    if kind == "layer":
        c.update(F=rng.choice(widths), F2=rng.choice(widths[:4]), relu=rng.random() < 0.5,
                 xbf16=rng.random() < 0.5, bf16=rng.random() < 0.5)
    if kind in ("forward", "train"):
        c.update(F=rng.choice(widths), F2=rng.choice(widths[:4]), F3=rng.choice([32, 64]),
                 xbf16=rng.random() < 0.5)
    if kind == "values":
        c["agg"] = rng.choice(["gcn", "mean", "sum"])
    return c


# ------------------------------------------------------------------ graphs

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + stream) & 0x7FFFFFFFFFFFFFFF)
    return g


def _rmat_edges(n, m, gen):
    """m distinct undirected edges (lo, hi) of an R-MAT graph (.57, .19, .19, .05), ids shuffled."""
    scale = max(1, (n - 1).bit_length())
    have = torch.empty(0, dtype=torch.int64, device=DEV)
    want = int(m * 1.3) + 1024
    while have.numel() < m:
        src = torch.zeros(want, dtype=torch.int64, device=DEV)
        dst = torch.zeros(want, dtype=torch.int64, device=DEV)
        for level in range(scale):
            r = torch.rand(want, device=DEV, generator=gen)
            low = r >= 0.76
            src |= low.long() << level
            dst |= ((r >= 0.57) ^ low ^ (r >= 0.95)).long() << level
        src, dst = (src * n) >> scale, (dst * n) >> scale
        keep = src != dst
        src, dst = src[keep], dst[keep]
        key = torch.minimum(src, dst) * n + torch.maximum(src, dst)
        have = torch.unique(torch.cat([have, key]))
        want = max(1024, int((m - have.numel()) * 2))
    have = have[torch.randperm(have.numel(), device=DEV, generator=gen)[:m]]
    relabel = torch.randperm(n, device=DEV, generator=gen)
    return relabel[torch.div(have, n, rounding_mode="floor")], relabel[have % n]


def _sbm_sizes(n):
    """Community sizes, log-uniform in 64..1024: fixed by n, about two thirds of the nodes."""
    r = np.random.RandomState(n & 0x7FFFFFFF)
    sizes, left = [], 2 * n // 3
    while left >= 64:
        s = min(left, int(64 * 16 ** r.random_sample()))
        sizes.append(s)
        left -= s
    return sizes


def _sbm_edges(n, m, gen):
    """Communities with p_in = 0.2 and about m bridges with Zipf end points (exponent 2.1)."""
    keys, off = [], 0
    for s in _sbm_sizes(n):
        ij = (torch.rand((s, s), device=DEV, generator=gen) < 0.2).triu_(1).nonzero()
        keys.append((ij[:, 0] + off) * n + ij[:, 1] + off)
        off += s
    rank = (torch.randperm(n, device=DEV, generator=gen) + 1).double()
    cdf = torch.cumsum(rank.pow(-1.0 / 1.1), 0)
    ends = torch.searchsorted(cdf / cdf[-1], torch.rand((2, m), device=DEV, generator=gen, dtype=torch.float64))
    a, b = ends.clamp_(max=n - 1)
    ok = a != b
    keys.append(torch.minimum(a, b)[ok] * n + torch.maximum(a, b)[ok])
    key = torch.unique(torch.cat(keys))
    return torch.div(key, n, rounding_mode="floor"), key % n


def _graph(case, seed):
    n = case["n"]
    gen = _gen(seed, 1)
    lo, hi = (_rmat_edges if case["graph"] == "rmat" else _sbm_edges)(n, case["m"], gen)
    loop = torch.arange(n, device=DEV)
    key = torch.cat([lo * n + hi, hi * n + lo, loop * (n + 1)]).sort().values
    row = torch.div(key, n, rounding_mode="floor")
    col = (key - row * n).int()
    deg = torch.bincount(row, minlength=n)
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    rowptr[1:] = torch.cumsum(deg, 0).int()
    val = (deg[row].double() * deg[col.long()].double()).rsqrt().float()
    return rowptr, col.contiguous(), val


def _randn(case, seed, stream, rows, cols):
    return torch.randn((rows, cols), device=DEV, generator=_gen(seed, stream))


def _glorot(seed, stream, fi, fo):
    a = math.sqrt(6.0 / (fi + fo))
    return (torch.rand((fi, fo), device=DEV, generator=_gen(seed, stream)) * 2 - 1) * a


def _inputs(case, seed):
    kind, n = case["kind"], case["n"]
    s = {"kind": kind, "case": case}
    s["rowptr"], s["col"], s["val"] = _graph(case, seed)
    if "F" in case:
        X = _randn(case, seed, 2, n, case["F"])
        s["X"] = X.to(torch.bfloat16) if case.get("xbf16") else X
    if "F2" in case:
        s["W1"] = _glorot(seed, 3, case["F"], case["F2"])
    if "F3" in case:
        s["W2"] = _glorot(seed, 4, case["F2"], case["F3"])
    if kind == "train":     # 10% of the rows carry a class
        gen = _gen(seed, 5)
        lab = torch.randint(0, case["F3"], (n,), device=DEV, generator=gen, dtype=torch.int32)
        lab[torch.rand(n, device=DEV, generator=gen) >= 0.1] = -1
        lab[0] = 0
        s["labels"] = lab
        s["scale"] = 1.0 / int((lab >= 0).sum().item())
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, n = case["kind"], case["n"]
    A = (s["rowptr"], s["col"], s["val"])
    if kind in ("spmm", "layer", "forward", "train"):
        s["plan"] = dg.Plan(*A, seed=0)
    if kind == "reload":
        s["kept"] = dg.Plan(*A, seed=0, walks_per_node=case["walks"], walk_len=case["steps"])

    def empty(cols, dtype=torch.float32):
        return torch.empty((n, cols), dtype=dtype, device=DEV)

    if kind in ("spmm", "layer"):
        s["Y"] = empty(case["F2"] if kind == "layer" else case["F"],
                       torch.bfloat16 if case["bf16"] else torch.float32)
    if kind in ("build", "reload"):
        s["Y"] = empty(case["F"])
    if kind == "layer":
        s["ws"] = torch.empty(dg.gcn_layer_workspace_bytes(s["plan"], case["F"], case["F2"]),
                              dtype=torch.uint8, device=DEV)
    if kind in ("forward", "train"):
        s["T1"], s["T2"], s["Y"] = empty(case["F2"]), empty(case["F3"]), empty(case["F3"])
        s["H1"] = empty(case["F2"], torch.bfloat16)
    if kind == "train":
        s["G"], s["loss"] = empty(case["F3"]), torch.empty(dg.LOSS_SLOTS, dtype=torch.float64, device=DEV)
        s["dT2"], s["dT1"] = empty(case["F3"], torch.bfloat16), empty(case["F2"], torch.bfloat16)
        s["dH1"] = empty(case["F2"])
        s["dW1"], s["dW2"] = torch.empty_like(s["W1"]), torch.empty_like(s["W2"])
        s["ws"] = torch.empty(max(dg.weight_grad_workspace_bytes(n, case["F"], case["F2"]),
                                  dg.weight_grad_workspace_bytes(n, case["F2"], case["F3"])),
                              dtype=torch.uint8, device=DEV)
    return s


def _plan_numbers(plan):
    i = plan.info()
    return [i["n_sparse"], i["kstar"], i["kmax"], i["max_degree"]]


def run(s):
    kind, case = s["kind"], s["case"]
    if kind == "spmm":
        return dg.spmm(s["plan"], s["X"], s["Y"], relu=case["relu"], out_bf16=case["bf16"])
    if kind == "layer":
        return dg.gcn_layer(s["plan"], s["X"], s["W1"], relu=case["relu"], Y=s["Y"], workspace=s["ws"],
                            out_bf16=case["bf16"])
    if kind == "values":
        return dg.aggregator_values(s["rowptr"], s["col"], case["agg"], eps=0.5)
    if kind == "build":
        s["plan"] = dg.Plan(s["rowptr"], s["col"], s["val"], seed=0, walks_per_node=case["walks"],
                            walk_len=case["steps"])
        return [dg.spmm(s["plan"], s["X"], s["Y"]), _plan_numbers(s["plan"])]
    if kind == "reload":
        blob = s["kept"].save()
        s["plan"] = dg.Plan.load(s["rowptr"], s["col"], s["val"], blob)
        return [dg.spmm(s["plan"], s["X"], s["Y"]), _plan_numbers(s["plan"])]
    plan = s["plan"]
    dg.update(s["X"], s["W1"], s["T1"])
    if kind == "forward":       # the fused junction where it pays, as the program's step does
        dg.spmm_update(plan, s["T1"], s["W2"], s["T2"], relu=True)
        return dg.spmm(plan, s["T2"], s["Y"])
    dg.spmm_update(plan, s["T1"], s["W2"], s["T2"], relu=True, H=s["H1"])
    dg.spmm(plan, s["T2"], s["Y"])
    dg.softmax_xent(s["Y"], s["labels"], s["scale"], s["G"], s["loss"])
    dg.spmm(plan, s["G"], s["dT2"], out_bf16=True)
    dg.backward_data(s["dT2"], s["W2"], s["H1"], s["dH1"])
    dg.weight_grad(s["H1"], s["dT2"], s["dW2"], workspace=s["ws"])
    dg.spmm(plan, s["dH1"], s["dT1"], out_bf16=True)
    dg.weight_grad(s["X"], s["dT1"], s["dW1"], workspace=s["ws"])
    return [s["Y"], s["loss"][0], s["dW1"], s["dW2"]]


# ------------------------------------------------------------------ what a pass cannot do without

def _nnz(case):
    if case["graph"] == "rmat":
        return 2 * case["m"] + case["n"]
    intra = sum(0.2 * z * (z - 1) / 2 for z in _sbm_sizes(case["n"]))
    return int(2 * intra + 2 * case["m"] + case["n"])


def work(case):
    n, nnz, kind = case["n"], _nnz(case), case["kind"]
    csr = 4 * (n + 1) + 8 * nnz
    F, F2, F3 = case.get("F", 0), case.get("F2", 0), case.get("F3", 0)
    xb = 2 if case.get("xbf16") else 4
    yb = 2 if case.get("bf16") else 4
    if kind == "values":
        return {"bytes": 4 * (n + 1) + 8 * nnz, "flops": 0}
    if kind in ("spmm", "build"):
        return {"bytes": csr + (4 + yb) * n * F, "flops": 2.0 * nnz * F}
    if kind == "reload":        # the density sums go to the host and back
        return {"bytes": csr + 8 * n * F + 8 * n, "flops": 2.0 * nnz * F}
    if kind == "layer":
        return {"bytes": csr + n * (xb * F + yb * F2), "flops": 2.0 * n * F * F2 + 2.0 * nnz * F2}
    if kind == "forward":
        return {"bytes": csr + n * (xb * F + 4 * F3),
                "flops": 2.0 * n * (F * F2 + F2 * F3) + 2.0 * nnz * (F2 + F3)}
    return {"bytes": csr + n * (xb * F + 4 * F3 + 4) + 4 * (F * F2 + F2 * F3),
            "flops": 2.0 * n * (2 * F * F2 + 3 * F2 * F3) + 4.0 * nnz * (F2 + F3)}


def tolerance(case):
    """About four times the distance from the 64-bit results that the path was measured at."""
    kind = case["kind"]
    if kind in ("spmm", "layer") and case["bf16"]:   # a bfloat16 output's last place: 1.7e-3
        return {"rel": 7e-3}
    if kind in ("spmm", "build", "reload", "values"):    # one rounding of a 64-bit sum: 2e-8
        return {"rel": 1e-7}
    if kind == "layer":         # 32-bit sums of the matrix cores, then the aggregation
        return {"rel": 1e-6}
    # a sum that rounds to the other bfloat16 between two layers: 2e-5 to 2.5e-5
    return {"rel": 1e-4}


# ------------------------------------------------------------------ 64-bit references

def _spmm64(s, X):
    """A X in float64, by blocks of entries."""
    n = s["rowptr"].numel() - 1
    row = torch.repeat_interleave(torch.arange(n, device=DEV), s["rowptr"].diff().long())
    Y = torch.zeros((n, X.shape[1]), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 28) // X.shape[1])
    for e in range(0, row.numel(), step):
        f = slice(e, e + step)
        part = X[s["col"][f].long()].double()
        Y.index_add_(0, row[f], part.mul_(s["val"][f].double().unsqueeze(1)))
    return Y


def _bf(x):
    """The bfloat16 rounding that the matrix-core products apply to their operands."""
    return x.float().to(torch.bfloat16).double()


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "values":
        deg = s["rowptr"].diff().double()
        n = case["n"]
        row = torch.repeat_interleave(torch.arange(n, device=DEV), s["rowptr"].diff().long())
        if case["agg"] == "gcn":
            return (deg[row] * deg[s["col"].long()]).rsqrt()
        if case["agg"] == "mean":
            return 1.0 / deg[row]
        return torch.where(row == s["col"], 1.5, 1.0).double()
    if kind == "spmm":
        Y = _spmm64(s, s["X"])
        return Y.relu() if case["relu"] else Y
    if kind in ("build", "reload"):
        return [_spmm64(s, s["X"]), None]
    T1 = _bf(s["X"]) @ _bf(s["W1"])
    if kind == "layer":
        Y = _spmm64(s, T1)
        return Y.relu() if case["relu"] else Y
    H1 = _bf(_spmm64(s, T1).relu())
    del T1
    W2 = _bf(s["W2"])
    Y = _spmm64(s, H1 @ W2)
    if kind == "forward":
        return Y
    lab = s["labels"].long()
    on = lab >= 0
    p = torch.log_softmax(Y[on], 1)
    hit = lab[on].unsqueeze(1)
    loss = -p.gather(1, hit).sum() * s["scale"]
    G = torch.zeros_like(Y)
    g = p.exp()
    g.scatter_add_(1, hit, torch.full_like(hit, -1, dtype=torch.float64))
    G[on] = g * s["scale"]
    dT2 = _bf(_spmm64(s, G))
    dW2 = H1.t().contiguous() @ dT2
    dH1 = torch.where(H1 > 0, dT2 @ W2.t().contiguous(), 0.0)
    dT1 = _bf(_spmm64(s, dH1))
    dW1 = _bf(s["X"]).t().contiguous() @ dT1
    return [Y, loss, dW1, dW2]
