"""Every way an SpMM launch requests its gathers: 32-bit offsets, cache classes and 64-bit
addresses; a round, half a round and a quarter of it at a time; whole rows and slices of 64
features; groups of 8, 16, 32 and 64 lanes.  Which one a launch takes goes by the operand's
size, the number of entries and the number of long rows, so the matrices here lie on both sides of
each bound.  None of it may change a result: every row is checked, fp32 within 1e-5 sum |a||x|
and bfloat16 after ReLU within a half unit in the last place more."""
import ctypes

import numpy as np
import pytest
import torch


from fullrows import act_bf16_judge, compare_all_rows, spmm_judge
from graphgen.csr import Graph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg(device):
    import paper_2609_01983_amd as dg
    return dg


def _matrix(n, entries, long_rows, seed):
    """About `entries` entries: empty and short rows, `long_rows` rows of 512 to 900 entries, one of
    5,000 and one of 13,000 (split into parts)."""
    gen = np.random.default_rng(seed)
    deg = gen.geometric(0.5, n) - 1                   # one entry a row on average
    at = gen.choice(n, long_rows + 2, replace=False)
    deg[at[:-2]] = gen.integers(512, 901, long_rows)
    deg[at[-2:]] = [5000, 13000]
    left = entries - int(deg.sum())
    deg += left // n if left > 0 else 0
    rowptr = np.zeros(n + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(deg)
    m = int(rowptr[-1])
    col = np.minimum(gen.integers(0, n, m), gen.integers(0, n, m)).astype(np.int32)     # low columns hot
    return Graph(n=n, rowptr=rowptr, col=col, val=gen.standard_normal(m).astype(np.float32))


# matrix: (nodes, entries, long rows), then widths
CASES = {
    # half rounds: many long rows, small operands
    "many_small": ((20000, 400000, 300), [33, 64, 100, 128, 130, 192, 200, 256]),
    # a round and, above 128 MiB, half: few long rows (F = 192 and 256 in slices, and whole)
    "few": ((130000, 700000, 20), [64, 100, 128, 168, 192, 200, 256]),
    "few_large": ((270001, 1300000, 20), [60, 128, 136, 192, 200]),
    # quarter rounds: many long rows, 88 to 256 MiB, enough entries for the parts' chains
    "deep": ((300007, 3000000, 300), [28, 78, 96, 120, 128, 132, 192, 200]),
    # the same operands, too few entries: half rounds
    "shallow": ((300007, 2400000, 300), [78, 120, 128, 200]),
    # cache classes (over 256 MiB): halves with four and five workgroups a CU, quarters
    "classes_deep": ((700001, 3300000, 300), [34, 60, 96, 97, 100, 128, 160, 192, 193, 200]),
    "classes_shallow": ((700001, 2400000, 300), [60, 100, 200]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_every_gather_variant(dg, device, name):
    (n, entries, long_rows), widths = CASES[name]
    g = _matrix(n, entries, long_rows, seed=n)
    A = (torch.from_numpy(g.rowptr).to(device), torch.from_numpy(g.col).to(device), torch.from_numpy(g.val).to(device))
    plan = dg.Plan(*A, seed=0, walks_per_node=4, walk_len=3)
    info = plan.info()
    cus = torch.cuda.get_device_properties(device).multi_processor_count
    assert (info["n_long_rows"] + info["n_split_parts"] <= cus) == name.startswith("few")
    assert info["n_split_rows"] > 0
    if name.endswith(("deep", "shallow")):
        assert (info["nnz"] >= 2560 * info["dense_chunk"]) == name.endswith("deep")
    assert info["cold_marked"] == int(n > 1 << 18)
    gen = torch.Generator(device=device).manual_seed(n)
    for F in widths:
        print(f"[gathers] {name} F={F}", flush=True)
        X = torch.randn((n, F), device=device, generator=gen)
        Xh = X.cpu().numpy()
        Y = dg.spmm(plan, X, torch.full((n, F), float("nan"), device=device))
        compare_all_rows(g, Xh, Y.cpu().numpy(), spmm_judge(), what=f"{name} F={F}")
        H = dg.spmm(plan, X, torch.full((n, F), float("nan"), dtype=torch.bfloat16, device=device), relu=True,
                    out_bf16=True)
        # the kernel's bfloat16 output is the rounding of the fp32 one
        assert torch.equal(H, torch.relu(Y).to(torch.bfloat16)), (name, F)
        if F % 32 == 0 and F <= 256:                  # the fused kernel, whatever the route
            W = torch.randn((F, 32), device=device, generator=gen) / F ** 0.5
            T = torch.full((n, 32), float("nan"), device=device)
            st = dg.lib().dualgcn_spmm_update(plan.handle, X.data_ptr(), W.data_ptr(), T.data_ptr(), None, F, 32,
                                              dg.RELU, ctypes.c_void_p(0))
            torch.cuda.synchronize()
            assert st == dg.OK
            assert torch.equal(T, dg.update(H, W)), (name, F)
    plan.destroy()


def _device_matrix(device, n, long_rows):
    """Rows of 0 to 3 entries, `long_rows` of 600 and one of 9,000, on the device."""
    gen = torch.Generator(device=device).manual_seed(n)
    deg = torch.randint(0, 4, (n,), device=device, generator=gen)
    at = torch.randperm(n, device=device, generator=gen)[:long_rows + 1]
    deg[at] = 600
    deg[at[0]] = 9000
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=device)
    rowptr[1:] = torch.cumsum(deg, 0)
    m = int(rowptr[-1])
    col = torch.randint(0, n, (m,), device=device, dtype=torch.int32, generator=gen)
    val = torch.randn(m, device=device, generator=gen)
    return rowptr.to(torch.int32), col, val


def _check_rows(A, X, Y, chunk=1 << 21):
    """Every row of Y within 1e-5 sum |a||x| of the float64 sums, computed entry by entry."""
    rowptr, col, val = A
    n = rowptr.numel() - 1
    for r0 in range(0, n, chunk):
        r1 = min(n, r0 + chunk)
        e0, e1 = int(rowptr[r0]), int(rowptr[r1])
        row = torch.repeat_interleave(torch.arange(r1 - r0, device=X.device), rowptr[r0:r1 + 1].diff().long())
        S = torch.zeros((r1 - r0, X.shape[1]), dtype=torch.float64, device=X.device)
        B = torch.zeros_like(S)
        step = max(1, (1 << 27) // X.shape[1])
        for e in range(e0, e1, step):
            f = slice(e, min(e1, e + step))
            P = X[col[f].long()].double() * val[f].double().unsqueeze(1)
            S.index_add_(0, row[f.start - e0:f.stop - e0], P)
            B.index_add_(0, row[f.start - e0:f.stop - e0], P.abs_())
        bad = ~((Y[r0:r1].double() - S).abs() <= 1e-5 * B)         # a NaN is bad
        assert not bool(bad.any()), (r0, int(bad.sum()))


@pytest.mark.parametrize("n,widths", [(4300000, [250, 260, 356, 512]), (8500000, [127, 128])])
def test_operands_of_more_than_four_gib(dg, device, n, widths):
    """64-bit addresses in groups of 64, 32, 16 lanes, in slices and in a window of one lane."""
    A = _device_matrix(device, n, 300)
    plan = dg.Plan(*A, seed=0, walks_per_node=2, walk_len=2)
    for F in widths:
        print(f"[wide] n={n} F={F}", flush=True)
        assert n * F * 4 > 0xFF800000
        X = torch.randn((n, F), device=device)
        Y = dg.spmm(plan, X, torch.full((n, F), float("nan"), device=device))
        _check_rows(A, X, Y)
        del X, Y
    plan.destroy()


def test_more_nodes_than_the_schedule_adds_directly(dg, device):
    """2^24 + 5,003 nodes: more than 4,096 schedule tiles, so their sums are scanned by a workgroup
    of its own; sparse tasks, long rows and split rows on every row of an aggregation (64-bit
    addresses in 16-lane groups) and of the fused junction."""
    n = (1 << 24) + 5003
    A = _device_matrix(device, n, 300)
    plan = dg.Plan(*A, seed=0, walks_per_node=2, walk_len=2)
    info = plan.info()
    deg = A[0].diff()
    chunk = info["dense_chunk"]
    split = deg[deg > chunk]
    assert info["n_split_rows"] == split.numel() and info["n_split_parts"] == int(((split + chunk - 1) // chunk).sum())
    perm = torch.from_numpy(plan.export()[0])
    assert torch.equal(perm.sort().values, torch.arange(n, dtype=torch.int32))
    X = torch.randn((n, 64), device=device)
    assert X.numel() * 4 > 0xFF800000
    Y = dg.spmm(plan, X, torch.full((n, 64), float("nan"), device=device))
    _check_rows(A, X, Y)
    del Y
    W = torch.randn((64, 32), device=device) / 8
    T = torch.full((n, 32), float("nan"), device=device)
    assert dg.spmm_update_route(plan, 64, 32)
    dg.spmm_update(plan, X, W, T, relu=True)
    assert torch.equal(T, dg.update(dg.spmm(plan, X, relu=True, out_bf16=True), W))
    plan.destroy()
