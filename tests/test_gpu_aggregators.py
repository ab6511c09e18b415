"""GPU parity of the aggregator values (GCN, mean, sum/GIN) and of the SpMM on them.

Values: float64 arithmetic rounded once to float32 on both sides; they may differ only
where the device square root is not correctly rounded, so the test allows one float32
ulp and reports how many values match exactly.  SpMM: the usual 1e-5 sum |a||x| bound.
"""
import time

import numpy as np
import pytest
import torch

import oracle
from graphgen import configs, dense, small
from graphgen.csr import Graph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg(device):
    import paper_2609_01983_amd as dg
    return dg


GRAPHS = {
    "star": lambda: small.star(300, self_loops=True),
    "gnp": lambda: small.random_graph(200, 0.05, seed=3),
    "rows": lambda: small.from_rows([[0, 1, 2], [1, 0], [2, 2, 0], [], [1], [5, 5, 5, 0]]),
    "c2": lambda: configs.load_graph("c2"),
}


def _dev(g, device):
    return (torch.from_numpy(np.ascontiguousarray(g.rowptr)).to(device),
            torch.from_numpy(np.ascontiguousarray(g.col)).to(device))


def _ulps(a, b):
    ai = a.view(np.int32).astype(np.int64)
    bi = b.view(np.int32).astype(np.int64)
    return np.abs(ai - bi)


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("kind,eps", [("gcn", 0.0), ("mean", 0.0), ("sum", 0.0), ("sum", 0.3)])
def test_aggregator_values(dg, device, name, kind, eps):
    g = GRAPHS[name]()
    rp, c = _dev(g, device)
    v = dg.aggregator_values(rp, c, kind, eps).cpu().numpy()
    ref = oracle.aggregator_values(g, {"gcn": oracle.AGG_GCN, "mean": oracle.AGG_MEAN,
                                       "sum": oracle.AGG_SUM}[kind], eps)
    finite = np.isfinite(ref)
    assert np.array_equal(np.isfinite(v), finite)
    assert _ulps(v[finite], ref[finite]).max(initial=0) <= 1
    if kind != "gcn":
        assert np.array_equal(v, ref)                 # one correctly rounded division


def _tiles(n, lengths, seed):
    """Rows of the given lengths (cycled) with random columns."""
    gen = np.random.default_rng(seed)
    return small.from_rows([gen.integers(0, n, lengths[i % len(lengths)]).tolist() for i in range(n)])


@pytest.mark.parametrize("n,lengths", [
    (1, [1]), (1, [2048]), (1, [2049]), (2, [2048, 1]), (3, [0, 4096, 0]), (700, [0, 0, 0, 7, 0]),
    (5000, [0] * 999 + [3]),        # tiles that meet more rows than entries
    (4097, [1]), (300, [0, 31, 5000, 1, 2]),
    (1 << 18, [1]), ((1 << 18) + 1, [1]),
    (300000, [0, 0, 5, 0, 9, 0]),             # tiles with empty rows
    (1, [300000]), (3, [5, 290000, 7]),       # a row of more tiles than its wavefront has lanes
    (70, [32768, 32769, 3]), (130, [0, 40000]),   # rows on both sides of 16 tiles, several a wavefront
    (1200000, [0] * 2999 + [1400])])          # tiles that meet more rows than entries
@pytest.mark.parametrize("kind", ["gcn", "mean", "sum"])
def test_aggregator_tiles(dg, device, n, lengths, kind):
    """Rows that start, end and span at the edges of the kernel's tiles of 2,048 entries."""
    g = _tiles(n, lengths, 5)
    rp, c = _dev(g, device)
    v = dg.aggregator_values(rp, c, kind, 0.25).cpu().numpy()
    ref = oracle.aggregator_values(g, {"gcn": oracle.AGG_GCN, "mean": oracle.AGG_MEAN,
                                       "sum": oracle.AGG_SUM}[kind], 0.25)
    finite = np.isfinite(ref)                       # a column whose own row is empty: 1 / 0
    assert np.array_equal(np.isfinite(v), finite)
    assert _ulps(v[finite], ref[finite]).max(initial=0) <= 1


@pytest.mark.parametrize("n,lengths", [
    (327680, [2]), (327681, [2]),              # 5 * 2^17 entries: the last searched, the next in tiles
    (1310719, [1]), (1310720, [1]),            # below and at 5 * 2^18 entries, as many rows
    (1400001, [0, 2]), (1966081, [1, 0, 1]),   # from there: up to 3/2 rows an entry in tiles (GCN)
    (5242881, [1, 0, 0, 0])])                  # up to 4 (the others)
@pytest.mark.parametrize("kind", ["gcn", "mean", "sum"])
def test_aggregator_search_and_tiles(dg, device, n, lengths, kind):
    """Values of matrices on both sides of the bounds between a search per entry and tiles."""
    deg = np.resize(np.array(lengths, dtype=np.int64), n)
    rowptr = np.zeros(n + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(deg)
    col = np.random.default_rng(9).integers(0, n, int(rowptr[-1])).astype(np.int32)
    col[::7] = np.repeat(np.arange(n), deg)[::7]          # diagonal entries
    g = Graph(n=n, rowptr=rowptr, col=col, val=np.ones(col.size, dtype=np.float32))
    rp, c = _dev(g, device)
    v = dg.aggregator_values(rp, c, kind, 0.25).cpu().numpy()
    with np.errstate(divide="ignore"):
        ref = oracle.aggregator_values(g, {"gcn": oracle.AGG_GCN, "mean": oracle.AGG_MEAN,
                                           "sum": oracle.AGG_SUM}[kind], 0.25)
    finite = np.isfinite(ref)
    assert np.array_equal(np.isfinite(v), finite)
    assert _ulps(v[finite], ref[finite]).max(initial=0) <= 1


@pytest.mark.parametrize("n,per_row", [(1000, 5), (1 << 16, 4), ((1 << 16) + 1, 4), (100000, 7)])
@pytest.mark.parametrize("kind", ["gcn", "mean", "sum"])
def test_row_pointers_out_of_order_leave_the_values_alone(dg, device, n, per_row, kind):
    """On both sides of the bound between the search per entry (up to 5 * 2^17 entries) and the tiles."""
    g = _tiles(n, [per_row], 7)
    rp, c = _dev(g, device)
    rp[n // 2] += 2 * per_row                         # within the entries, above its successor
    val = torch.full((c.numel(),), 7.0, device=device)
    with pytest.raises(dg.DualGCNError) as e:
        dg.aggregator_values(rp, c, kind, val=val)
    assert e.value.status == dg.ERR_BAD_CSR
    assert torch.all(val == 7.0)


def _ms(call):
    """Shortest of ten calls, each waited for."""
    best = float("inf")
    for _ in range(10):
        torch.cuda.synchronize()
        t = time.perf_counter()
        call()
        torch.cuda.synchronize()
        best = min(best, 1e3 * (time.perf_counter() - t))
    return best


def test_one_row_of_all_entries_costs_no_more_than_short_rows(dg, device):
    """2^24 entries in rows of 64, and all of them in one row of the same nodes: the same bytes.
    One thread that wrote all tile ends of the row took the call to three times as long."""
    n, m = 1 << 18, 1 << 24
    gen = torch.Generator(device=device).manual_seed(3)
    col = torch.randint(0, n, (m,), device=device, dtype=torch.int32, generator=gen)
    spread = (torch.arange(n + 1, device=device) * (m // n)).to(torch.int32)
    one = torch.zeros(n + 1, dtype=torch.int32, device=device)
    one[n // 3:] = m
    val = torch.empty(m, dtype=torch.float32, device=device)
    times = [_ms(lambda: dg.aggregator_values(rp, col, "mean", val=val)) for rp in (spread, one)]
    assert times[1] <= 1.6 * times[0], times
    assert torch.all(val == torch.tensor(1.0 / m, dtype=torch.float64).float().item())


@pytest.mark.parametrize("kind", ["mean", "sum"])
def test_spmm_with_other_aggregators_c2(dg, device, kind):
    g = configs.load_graph("c2")
    w = configs.WORKLOADS["c2"]
    rp, c = _dev(g, device)
    val = dg.aggregator_values(rp, c, kind, 0.1)
    plan = dg.Plan(rp, c, val, seed=0, walks_per_node=w.walks, walk_len=w.steps)
    X = dense.features_normal(g.n, 64, seed=4)
    Y = dg.spmm(plan, torch.from_numpy(X).to(device)).cpu().numpy()
    gv = type(g)(n=g.n, rowptr=g.rowptr, col=g.col, val=val.cpu().numpy())
    Yr, B = oracle.spmm(gv, X)
    assert np.all(np.abs(Y - Yr) <= 1e-5 * B)


def test_aggregator_rejects_bad_csr(dg, device):
    g = small.random_graph(20, 0.2, seed=3)
    rp, c = _dev(g, device)
    c = c.clone()
    c[2] = 99
    with pytest.raises(dg.DualGCNError) as e:
        dg.aggregator_values(rp, c, "gcn")
    assert e.value.status == dg.ERR_BAD_CSR
