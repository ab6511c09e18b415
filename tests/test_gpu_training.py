"""GPU parity of the training path: the HIP kernels (through the C ABI) against the
oracle's float64 chain rule.

* softmax cross-entropy: G within 1e-5 * scale per element, the loss within 1e-5 of
  scale * sum |terms|;
* weight gradient and backward data (bf16 matrix cores): within 1e-2 * (|X|^T |G|)
  and 1e-2 * (|G| |W|^T) per element, masks exact;
* the transposed aggregation on a plan of A^T: the SpMM bound 1e-5 * sum |a||g|;
* a whole two-layer training step on the c2 graph: within bounds propagated through
  the chain from the per-stage budgets above, and within 1e-3 (normwise) of the same
  chain computed with the declared bfloat16 roundings in float64.
"""
import numpy as np
import pytest
import torch

import oracle
import trainbound
from graphgen import configs, dense, small
from graphgen.csr import transposed

pytestmark = pytest.mark.gpu

BF16_TOL = 1e-2


@pytest.fixture(scope="module")
def dg(device):
    import paper_2609_01983_amd as dg
    return dg


def to_dev(g, device):
    return (torch.from_numpy(np.ascontiguousarray(g.rowptr)).to(device),
            torch.from_numpy(np.ascontiguousarray(g.col)).to(device),
            torch.from_numpy(np.ascontiguousarray(g.val)).to(device))


def _bf16_values(a):
    """float32 array of the bfloat16 values torch stores for `a` (the test's own rounding,
    used only to build inputs)."""
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(torch.bfloat16).float().numpy()


def _within(got, want, bound, tol, what):
    got = np.asarray(got, dtype=np.float64)
    err = np.abs(got - want)
    bad = ~(err <= tol * bound)
    if bad.any():
        i = tuple(np.argwhere(bad)[0])
        raise AssertionError(f"{what}: {bad.sum()} outside; first at {i}: got {got[i]!r} "
                             f"want {want[i]!r} bound {bound[i]!r}")


# ---------------------------------------------------------------- softmax cross-entropy

def _labels(n, C, seed):
    y = dense.labels(n, C, seed, labeled_fraction=0.7)
    y[::97] = C + 3                                   # out of range: unlabeled as well
    return y


@pytest.mark.parametrize("n,C", [(1, 1), (300, 3), (1000, 16), (777, 17), (4096, 64), (513, 100)])
def test_softmax_xent(dg, device, n, C):
    Y = dense.features_normal(n, C, seed=n + C) * np.float32(3.0)
    labels = _labels(n, C, seed=C)
    scale = 1.0 / max(1, int(((labels >= 0) & (labels < C)).sum()))
    G, loss = dg.softmax_xent(torch.from_numpy(Y).to(device), torch.from_numpy(labels).to(device),
                              scale)
    ref_loss, ref_G = oracle.softmax_xent(Y, labels, scale)
    _within(G.cpu().numpy(), ref_G, np.full(ref_G.shape, scale), 1e-5, "G")
    assert abs(loss[0].item() - ref_loss) <= 1e-5 * trainbound.loss_bound(Y, labels, scale)
    # unlabeled rows get exactly zero gradient
    off = (labels < 0) | (labels >= C)
    assert np.all(G.cpu().numpy()[off] == 0.0)
    # bit-reproducible
    G2, loss2 = dg.softmax_xent(torch.from_numpy(Y).to(device), torch.from_numpy(labels).to(device),
                                scale)
    assert torch.equal(G, G2) and loss[0].item() == loss2[0].item()


@pytest.mark.parametrize("n,C", [(1000, 16), (777, 17), (4096, 64), (513, 100)])
def test_softmax_xent_unlabeled_logits_do_not_matter(dg, device, n, C):
    """The loss and its gradient depend on labeled rows only: logits of unlabeled rows
    replaced by NaN and infinities give the same G and loss bits (the vectorised and the
    scalar kernel do not read them)."""
    Y = dense.features_normal(n, C, seed=n + 2 * C) * np.float32(3.0)
    labels = _labels(n, C, seed=C + 1)
    scale = 1.0 / max(1, int(((labels >= 0) & (labels < C)).sum()))
    off = (labels < 0) | (labels >= C)
    Yb = Y.copy()
    Yb[off] = np.float32(np.nan)
    Yb[off, ::3] = np.float32(np.inf)
    Yb[off, 1::3] = np.float32(-np.inf)
    lab = torch.from_numpy(labels).to(device)
    G, loss = dg.softmax_xent(torch.from_numpy(Y).to(device), lab, scale)
    Gb, lossb = dg.softmax_xent(torch.from_numpy(Yb).to(device), lab, scale)
    assert torch.equal(G, Gb) and loss[0].item() == lossb[0].item()


def test_softmax_xent_c5_shape(dg, device):
    """The last layer of c5: n = 2^22 rows of 64 classes; every G row sampled, the loss whole."""
    n, C = 1 << 22, 64
    Y = dense.features_normal(n, C, seed=5, stream_id=7)
    labels = _labels(n, C, seed=5)
    scale = 1.0 / max(1, int(((labels >= 0) & (labels < C)).sum()))
    G, loss = dg.softmax_xent(torch.from_numpy(Y).to(device), torch.from_numpy(labels).to(device),
                              scale)
    Gh = G.cpu().numpy()
    rows = np.random.default_rng(1).choice(n, 4096, replace=False)
    rows = np.concatenate([rows, [0, n - 1]])
    _, ref_G = oracle.softmax_xent(Y[rows], labels[rows], scale)
    _within(Gh[rows], ref_G, np.full(ref_G.shape, scale), 1e-5, "G sampled")
    total = 0.0
    for lo in range(0, n, 1 << 20):
        total += oracle.softmax_xent(Y[lo:lo + (1 << 20)], labels[lo:lo + (1 << 20)], scale)[0]
    assert abs(loss[0].item() - total) <= 1e-5 * trainbound.loss_bound(Y, labels, scale)


# ---------------------------------------------------------------- weight gradient

@pytest.mark.parametrize("n,fin,fout", [(1, 32, 32), (64, 32, 32), (1000, 32, 64), (4133, 256, 128),
                                        (777, 128, 64), (2050, 1024, 256), (300, 96, 160),
                                        (129, 512, 32)])
@pytest.mark.parametrize("xbf,gbf", [(False, False), (True, True), (False, True), (True, False)])
def test_weight_grad(dg, device, n, fin, fout, xbf, gbf):
    X = dense.features_normal(n, fin, seed=fin + n)
    G = dense.features_normal(n, fout, seed=fout + 7, stream_id=7)
    Xt = torch.from_numpy(X).to(device)
    Gt = torch.from_numpy(G).to(device)
    if xbf:
        Xt = Xt.to(torch.bfloat16)
        X = _bf16_values(X)
    if gbf:
        Gt = Gt.to(torch.bfloat16)
        G = _bf16_values(G)
    dW = dg.weight_grad(Xt, Gt).cpu().numpy()
    ref, B = oracle.weight_grad(X, G)
    _within(dW, ref, B, BF16_TOL, f"dW {n}x{fin}x{fout}")
    _check_rounded_operands(dW, X, G)
    again = dg.weight_grad(Xt, Gt).cpu().numpy()
    assert np.array_equal(dW, again)


@pytest.mark.parametrize("partials", [120, 121, 128, 129, 137, 256])
@pytest.mark.parametrize("fin,fout", [(32, 32), (256, 256), (256, 224)])
def test_weight_grad_partial_counts(dg, device, partials, fin, fout):
    """Partial counts on both sides of whole batches of an eighth (16 at a time, and 4 from 2^16
    elements: 256 -> 256), ragged last chunk."""
    n = 64 * partials - 5
    X = _bf16_values(dense.features_normal(n, fin, seed=fin + n))
    G = _bf16_values(dense.features_normal(n, fout, seed=fout + 7, stream_id=7))
    dW = dg.weight_grad(torch.from_numpy(X).to(device).to(torch.bfloat16),
                        torch.from_numpy(G).to(device).to(torch.bfloat16)).cpu().numpy()
    _check_rounded_operands(dW, X, G)


def _check_rounded_operands(dW, X, G):
    """Against the exact product of the bfloat16 operands: only float32 accumulation is
    left, at most (rows per partial / 32 + 34) 2^-24 of sum |x||g| with at most 2^13 rows
    per partial below n = 2^22; 1e-4 of that sum covers it, and normwise 1e-4."""
    Xr, Gr = _bf16_values(X), _bf16_values(G)
    ref, B = oracle.weight_grad(Xr, Gr)
    _within(dW, ref, B, 1e-4, "dW vs bf16 operands")
    assert np.linalg.norm(dW - ref) <= 1e-4 * np.linalg.norm(ref) + 1e-30


def test_weight_grad_sgd_step(dg, device):
    n, fin, fout = 3000, 128, 64
    X = torch.from_numpy(dense.features_normal(n, fin, seed=1)).to(device)
    G = torch.from_numpy(dense.features_normal(n, fout, seed=2, stream_id=7)).to(device)
    W0 = torch.from_numpy(dense.glorot(fin, fout, seed=3)).to(device)
    W = W0.clone()
    dW = dg.weight_grad(X, G, lr=0.05, W=W)
    want = (W0.double() - 0.05 * dW.double()).cpu().numpy()
    got = W.double().cpu().numpy()
    assert np.all(np.abs(got - want) <= 1e-7 * (np.abs(want) + 0.05 * np.abs(dW.double().cpu().numpy())))


def test_weight_grad_c5_layer1_shape(dg, device):
    """dW1 at c5's shape (n = 2^22, 256 -> 128), X as the c5 features, G seeded."""
    n, fin, fout = 1 << 22, 256, 128
    X = dense.features_normal(n, fin, seed=0)
    G = _bf16_values(dense.features_normal(n, fout, seed=9, stream_id=7) * np.float32(1e-3))
    dW = dg.weight_grad(torch.from_numpy(X).to(device),
                        torch.from_numpy(G).to(device).to(torch.bfloat16)).cpu().numpy()
    ref = np.zeros((fin, fout))
    B = np.zeros((fin, fout))
    refr = np.zeros((fin, fout))
    Br = np.zeros((fin, fout))
    for lo in range(0, n, 1 << 19):
        Xc, Gc = X[lo:lo + (1 << 19)], G[lo:lo + (1 << 19)]
        r, b = oracle.weight_grad(Xc, Gc)
        ref += r
        B += b
        r, b = oracle.weight_grad(_bf16_values(Xc), Gc)
        refr += r
        Br += b
    _within(dW, ref, B, BF16_TOL, "dW c5 layer 1")
    _within(dW, refr, Br, 1e-4, "dW c5 layer 1 vs bf16 operands")
    assert np.linalg.norm(dW - refr) <= 1e-4 * np.linalg.norm(refr)
    # the bfloat16 copy of X (both operands bfloat16: the transposing-read kernel) gives
    # the same bits
    dWb = dg.weight_grad(torch.from_numpy(X).to(device).to(torch.bfloat16),
                         torch.from_numpy(G).to(device).to(torch.bfloat16)).cpu().numpy()
    assert np.array_equal(dWb, dW)


@pytest.mark.parametrize("n,fin,fout", [(1, 32, 32), (64, 32, 32), (4133, 256, 128), (777, 128, 64),
                                        (2050, 1024, 256), (300, 96, 160), (129, 512, 32),
                                        (70001, 224, 96)])
def test_weight_grad_operand_types_give_the_same_bits(dg, device, n, fin, fout):
    """Every operand is rounded to bfloat16 before the matrix cores, and every kernel takes
    the same chunks, k-steps and order of accumulation: passing X or G already rounded to
    bfloat16 (the kernel for two bfloat16 operands reads LDS with transposing reads) gives
    the same bits as passing them in float32."""
    X = torch.from_numpy(dense.features_normal(n, fin, seed=fin + 3 * n)).to(device)
    G = torch.from_numpy(dense.features_normal(n, fout, seed=fout + 5, stream_id=7)).to(device)
    want = dg.weight_grad(X, G)
    for xa, ga in ((X.to(torch.bfloat16), G), (X, G.to(torch.bfloat16)),
                   (X.to(torch.bfloat16), G.to(torch.bfloat16))):
        assert torch.equal(dg.weight_grad(xa, ga), want), (xa.dtype, ga.dtype)


# ---------------------------------------------------------------- backward data

@pytest.mark.parametrize("n,fin,fout", [(1, 32, 32), (1000, 64, 32), (4133, 256, 128), (777, 128, 64),
                                        (500, 1024, 64), (300, 96, 160), (65, 32, 256)])
@pytest.mark.parametrize("mask", [None, "f32", "bf16"])
@pytest.mark.parametrize("gbf", [False, True])
def test_backward_data(dg, device, n, fin, fout, mask, gbf):
    G = dense.features_normal(n, fout, seed=fout, stream_id=7)
    W = dense.glorot(fin, fout, seed=fin)
    Gt = torch.from_numpy(G).to(device)
    if gbf:
        Gt = Gt.to(torch.bfloat16)
        G = _bf16_values(G)
    M = Mt = None
    if mask is not None:
        M = dense.features_normal(n, fin, seed=3, stream_id=6)
        M[::5] = 0.0                                   # zeros are masked, like negatives
        Mt = torch.from_numpy(M).to(device)
        if mask == "bf16":
            Mt = Mt.to(torch.bfloat16)
            M = _bf16_values(M)
    dX = dg.backward_data(Gt, torch.from_numpy(W).to(device), Mt).cpu().numpy()
    ref, B = oracle.backward_data(G, W, M)
    _within(dX, ref, B, BF16_TOL, f"dX {n}x{fin}x{fout} mask={mask}")
    # exact product of the bfloat16 operands: float32 sums over F_out <= 256 terms only
    ref, B = oracle.backward_data(_bf16_values(G), _bf16_values(W), M)
    _within(dX, ref, B, 1e-5, f"dX vs bf16 operands {n}x{fin}x{fout}")
    if M is not None:
        assert np.all(dX[M <= 0] == 0.0)


# ---------------------------------------------------------------- transposed aggregation

def test_transposed_aggregation_on_plan_of_transpose(dg, device):
    rs = np.random.default_rng(3)
    rows = [list(rs.choice(400, size=rs.integers(0, 30), replace=True)) for _ in range(400)]
    rows[7] = list(range(400)) * 3                    # a hub row with duplicates
    g = small.from_rows(rows)
    g.val[:] = rs.uniform(-1, 1, g.col.size).astype(np.float32)
    gt = transposed(g)
    plan_t = dg.Plan(*to_dev(gt, device), seed=1, walks_per_node=8, walk_len=4)
    G = dense.features_normal(400, 48, seed=2, stream_id=7)
    got = dg.spmm(plan_t, torch.from_numpy(G).to(device)).cpu().numpy()
    want = oracle.spmm_f64(oracle.transpose_csr(g), G)
    gabs = small.from_rows(rows)
    gabs.val[:] = np.abs(g.val)
    B = oracle.spmm_f64(oracle.transpose_csr(gabs), np.abs(G))
    _within(got, want, B, 1e-5, "A^T G")


# ---------------------------------------------------------------- whole training step



def test_two_layer_training_step_c2(dg, device):
    g = configs.load_graph("c2")
    w = configs.WORKLOADS["c2"]
    X = configs.load_features("c2")
    F0, F1, C = X.shape[1], 32, 32
    W1 = dense.glorot(F0, F1, seed=0)
    W2 = dense.glorot(F1, C, seed=0, stream_id=5)
    labels = dense.labels(g.n, C, seed=0, labeled_fraction=0.1)
    scale = 1.0 / int((labels >= 0).sum())
    plan = dg.Plan(*to_dev(g, device), seed=0, walks_per_node=w.walks, walk_len=w.steps)
    Xd = torch.from_numpy(X).to(device)
    W1d = torch.from_numpy(W1).to(device)
    W2d = torch.from_numpy(W2).to(device)
    ld = torch.from_numpy(labels).to(device)
    # forward
    T1 = dg.update(Xd, W1d)
    H1 = dg.spmm(plan, T1, relu=True, out_bf16=True)
    T2 = dg.update(H1, W2d)
    Y2 = dg.spmm(plan, T2)
    # loss and backward
    G2, loss = dg.softmax_xent(Y2, ld, scale)
    dT2 = dg.spmm(plan, G2, out_bf16=True)
    dW2 = dg.weight_grad(H1, dT2).cpu().numpy()
    dH1 = dg.backward_data(dT2, W2d, H1)
    dT1 = dg.spmm(plan, dH1, out_bf16=True)
    dW1 = dg.weight_grad(Xd, dT1).cpu().numpy()

    ref = oracle.gcn_train_grads(g, X, [W1, W2], labels, scale)
    # error budgets propagated through the chain (float64, with |A| for every aggregation)
    E_loss, (E_dW1, E_dW2) = trainbound.two_layer_bounds(g, X, [W1, W2], labels, scale, ref)
    assert abs(loss[0].item() - ref["loss"]) <= E_loss
    _within(dW2, ref["dW"][1], E_dW2, 1.0, "dW2")
    _within(dW1, ref["dW"][0], E_dW1, 1.0, "dW1")
    # Those bounds hold whatever the signs, so over the n-row sums of dW they are loose.
    # Tight: the same chain with the declared bfloat16 roundings (operands of every dense
    # product, stored hidden activations and aggregated gradients) and float64 elsewhere
    # leaves only float32 summation and the rare bfloat16 tie on the other side: 1e-3
    # normwise, 1e-5 on the loss.
    ref16 = oracle.gcn_train_grads(g, X, [W1, W2], labels, scale, bf16=True)
    for got, want in ((dW1, ref16["dW"][0]), (dW2, ref16["dW"][1])):
        assert np.linalg.norm(got - want) <= 1e-3 * np.linalg.norm(want)
    assert abs(loss[0].item() - ref16["loss"]) <= 1e-5 * abs(ref16["loss"])


def test_label_restricted_plan_gives_the_loss_gradient_aggregation(dg, device):
    """The loss gradient vanishes on unlabeled rows, so A^T G = A G (A symmetric) needs only
    the entries whose column is labeled: the column-restricted matrix's own plan gives the
    same aggregation (the bench's training step uses it for the last layer)."""
    g = configs.load_graph("c2")
    w = configs.WORKLOADS["c2"]
    labels = dense.labels(g.n, 32, seed=3, labeled_fraction=0.1)
    Y = dense.features_normal(g.n, 32, seed=4)
    scale = 1.0 / int((labels >= 0).sum())
    _, G = oracle.softmax_xent(Y, labels, scale)
    keep = (labels >= 0)[g.col]
    rowptr_l = np.concatenate([[0], np.cumsum(keep)])[g.rowptr].astype(np.int32)
    gl = type(g)(n=g.n, rowptr=rowptr_l, col=g.col[keep].copy(), val=g.val[keep].copy())
    plan_l = dg.Plan(*to_dev(gl, device), seed=0, walks_per_node=w.walks, walk_len=w.steps)
    got = dg.spmm(plan_l, torch.from_numpy(G.astype(np.float32)).to(device)).cpu().numpy()
    want = oracle.spmm_f64(oracle.transpose_csr(g), G)
    ga = type(g)(n=g.n, rowptr=g.rowptr, col=g.col, val=np.abs(g.val))
    B = oracle.spmm_f64(oracle.transpose_csr(ga), np.abs(G))
    _within(got, want, B, 1e-5, "label-restricted A^T G")


def test_row_restricted_plan_gives_the_labeled_outputs(dg, device):
    """The loss reads the last layer's output on labeled rows only: the plan of the
    row-restricted matrix (unlabeled rows empty) gives those rows, and zeros elsewhere."""
    g = configs.load_graph("c2")
    w = configs.WORKLOADS["c2"]
    labels = dense.labels(g.n, 32, seed=5, labeled_fraction=0.1)
    lab = labels >= 0
    deg = np.diff(g.rowptr) * lab
    rowptr_r = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    keep = np.repeat(lab, np.diff(g.rowptr))
    gr = type(g)(n=g.n, rowptr=rowptr_r, col=g.col[keep].copy(), val=g.val[keep].copy())
    plan_r = dg.Plan(*to_dev(gr, device), seed=0, walks_per_node=w.walks, walk_len=w.steps)
    T = dense.features_normal(g.n, 32, seed=6)
    got = dg.spmm(plan_r, torch.from_numpy(T).to(device)).cpu().numpy()
    rows = np.flatnonzero(lab).astype(np.int32)
    want, B = oracle.spmm(g, T, rows)
    _within(got[rows], want, B, 1e-5, "row-restricted A T on labeled rows")
    assert np.all(got[~lab] == 0.0)
