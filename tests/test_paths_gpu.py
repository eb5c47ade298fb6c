"""Kernel paths chosen by size, at the sizes where they can go wrong, against the oracle and, where
two paths must agree bit for bit, against each other."""
import numpy as np
import pytest
import torch

from oracle import eh_oracle as O
from workloads import generators as G
from tests import parity_util as P

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def B():
    from paper_2407_21082_amd import binding
    return binding


def _ints(*shape):
    return torch.full(shape, -7, dtype=torch.int32, device=DEV)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows", [2, 3, 4, 5, 8, 13, 16])
def test_few_rows_cascade_is_row_by_row(B, dtype, rows):
    """The exchange of the kernel for at most 16 rows looks at four rows of a head at a time and
    its LayerNorm is dealt to three waves: full and partly filled turns of both, with rows leaving
    on the way.  A row's statistics do not depend on its neighbours, so the same row alone gives
    the same bits."""
    w = G.Workload("few", d=192, V=6000, n_heads=6, rows=rows, dtype=dtype, seed=70 + rows, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    full = P.oracle_all_heads(heads, hid.h, dtype == "bf16")
    tau = G.tau_for_schedule(full[0], w.n_heads)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows)
    ex, tok, H = _ints(rows), _ints(rows), torch.zeros((w.n_heads, rows), device=DEV)
    B.eh_cascade(ctx, hid.h, rows, ex, tok, H)
    B.eh_check(ctx)
    P.compare_cascade(f"few{rows}", ex, tok, H, full[0], full[2], full[3], tau, [])
    for r in range(rows):
        ex1, tok1, H1 = _ints(1), _ints(1), torch.zeros((w.n_heads, 1), device=DEV)
        B.eh_cascade(ctx, hid.h[:, r:r + 1], 1, ex1, tok1, H1)
        B.eh_check(ctx)
        assert int(ex1) == int(ex[r]) and int(tok1) == int(tok[r])
        assert torch.equal(H1[:, 0].view(torch.int32), H[:, r].view(torch.int32))
    B.eh_destroy(ctx)


def _eval(B, ctx, head, h, rows, **kw):
    H, lse, am = torch.zeros(rows, device=DEV), torch.zeros(rows, device=DEV), _ints(rows)
    B.eh_eval(ctx, head, h, rows, H, lse, am, **kw)
    torch.cuda.synchronize()
    return H, lse, am


@pytest.mark.parametrize("dtype,bias,V,d,R", [
    ("bf16", False, 5000, 96, 17), ("bf16", False, 4099, 160, 32), ("bf16", False, 4100, 1000, 33), ("bf16", False, 57000, 64, 64),
    ("bf16", False, 33, 8, 40), ("bf16", True, 1, 64, 3), ("bf16", True, 777, 136, 1), ("bf16", True, 4099, 96, 65),
    ("bf16", True, 60001, 32, 20), ("bf16", True, 1500, 264, 130), ("f32", False, 4099, 100, 17), ("f32", False, 777, 36, 32),
    ("f32", False, 60001, 16, 18), ("f32", True, 4100, 1028, 5), ("f32", True, 50, 4, 64), ("f32", True, 1500, 132, 97)])
def test_ksplit_projection(B, dtype, bias, V, d, R):
    """The kernel that splits the weight stream over k: odd and missing k-steps of its four waves,
    one and two blocks of 32 rows, ragged vocabulary slices, several passes per slice (V above
    57344), several groups of 64 rows; gathered rows and a live count on the device."""
    w = G.Workload("ks", d=d, V=V, n_heads=2, rows=R, dtype=dtype, seed=V + d + R)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    gen = torch.Generator(device=DEV).manual_seed(V + R)
    bs = [torch.randn(V, generator=gen, device=DEV) for _ in range(2)] if bias else None
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0, 0.0], max_rows=R, bias=bs)
    for l in range(2):
        W = P.f64(heads.W[l])
        orc = _oracle(hid.h[l], heads.gamma[l], heads.beta[l], W, bs[l] if bias else None, dtype == "bf16")
        got = _eval(B, ctx, l, hid.h[l], R)
        P.compare_head(f"ks{l}", *got, orc, [])
        # half of the rows, gathered backwards, the count on the device: the same bits, the rest untouched
        n = (R + 1) // 2
        if R <= 16 and not bias:
            continue
        idx = torch.arange(R - 1, -1, -1, dtype=torch.int32, device=DEV)
        sub = _eval(B, ctx, l, hid.h[l], R, row_idx=idx, n_rows_dev=torch.tensor([n], dtype=torch.int32, device=DEV))
        for a, b, left in zip(sub, got, (0.0, 0.0, -7)):
            assert torch.equal(a[:n], b.flip(0)[:n])
            assert bool((a[n:] == left).all())
    B.eh_destroy(ctx)


def _oracle(h, gamma, beta, W, bias, bf16):
    y = O.layernorm(P.f64(h), P.f64(gamma), P.f64(beta), 1e-5, bf16_out=bf16)
    z = y @ W.T + (0.0 if bias is None else P.f64(bias))
    m = z.max(axis=1, keepdims=True)
    S = np.exp(z - m).sum(axis=1)
    lse = m[:, 0] + np.log(S)
    p = np.exp(z - lse[:, None])
    top = np.sort(z, axis=1)
    gap = top[:, -1] - top[:, -2] if z.shape[1] > 1 else np.full(z.shape[0], np.inf)
    return lse - (p * z).sum(axis=1), lse, z.argmax(axis=1), gap


@pytest.mark.parametrize("rows", [17, 40, 64])
def test_many_heads_of_a_few_rows_in_one_stream(B, rows):
    """eh_eval_heads up to 64 rows (V up to 49152) walks the heads in one launch whose weight stream runs on from
    head to head: the same bits as a head at a time."""
    w = G.Workload("ksheads", d=224, V=9001, n_heads=5, rows=rows, dtype="bf16", seed=rows)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0] * 5, max_rows=rows)
    H, lse, am = torch.zeros((4, rows), device=DEV), torch.zeros((4, rows), device=DEV), _ints(4, rows)
    B.eh_eval_heads(ctx, 1, 4, hid.h[1:], rows, H, lse, am)
    for l in range(4):
        for a, b in zip(_eval(B, ctx, 1 + l, hid.h[1 + l], rows), (H[l], lse[l], am[l])):
            assert torch.equal(a, b)
    B.eh_destroy(ctx)


@pytest.mark.parametrize("dtype,rows", [("bf16", 9), ("bf16", 90), ("f32", 20)])
def test_cascade_of_heads_with_a_bias_vector(B, dtype, rows):
    """Heads with a bias vector run the two-launches-per-head cascade at every row count."""
    w = G.Workload("biascascade", d=128, V=3001, n_heads=5, rows=rows, dtype=dtype, seed=rows, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    bs = [0.3 * torch.randn(w.V, device=DEV) for _ in range(5)]
    full = [_oracle(hid.h[l], heads.gamma[l], heads.beta[l], P.f64(heads.W[l]), bs[l], dtype == "bf16") for l in range(5)]
    full = [np.stack([f[i] for f in full]) for i in range(4)]
    tau = G.tau_for_schedule(full[0], 5)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows, bias=bs)
    ex, tok, H, nev = _ints(rows), _ints(rows), torch.zeros((5, rows), device=DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    B.eh_cascade(ctx, hid.h, rows, ex, tok, H, nev)
    torch.cuda.synchronize()
    P.compare_cascade("biascascade", ex, tok, H, full[0], full[2], full[3], tau, [])
    assert int(nev) == int((ex.long() + 1).sum())
    B.eh_destroy(ctx)


@pytest.mark.parametrize("rows,V,d", [(20, 3000, 256), (32, 1000, 96), (33, 9000, 8), (40, 60001, 64), (64, 5000, 1000), (64, 4200, 32)])
def test_persistent_cascade_and_verification_up_to_64_rows(B, rows, V, d):
    """The persistent kernel on the k-split stream: one and two blocks of 32 rows, workgroups without a
    tile of their own (fewer than 244 tiles of 16), several passes per slice, as few as one k-step,
    rows leaving on the way; then the verification of the same rows by the same kernel."""
    w = G.Workload("rowsks", d=d, V=V, n_heads=5, rows=rows, dtype="bf16", seed=rows + V, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    full = P.oracle_all_heads(heads, hid.h, True)
    tau = G.tau_for_schedule(full[0], 5)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows)
    for _ in range(3):
        ex, tok, H = _ints(rows), _ints(rows), torch.zeros((5, rows), device=DEV)
        nev = torch.zeros(1, dtype=torch.int64, device=DEV)
        B.eh_cascade(ctx, hid.h, rows, ex, tok, H, nev)
        B.eh_check(ctx)
        P.compare_cascade("rowsks", ex, tok, H, full[0], full[2], full[3], tau, [])
        assert int(nev) == int((ex.long() + 1).sum())
    if rows <= 16 or rows % 4:
        return B.eh_destroy(ctx)
    k, Bsz = 3, rows // 4
    want = torch.tensor(full[2][4].reshape(Bsz, 4), dtype=torch.int32, device=DEV)
    draft = want[:, :k].contiguous()
    draft[1::2, 1] = (draft[1::2, 1] + 1) % V
    acc, nxt, tgt = _ints(Bsz), _ints(Bsz), _ints(Bsz, 4)
    B.dssd_verify(ctx, hid.h[4].reshape(Bsz, 4, d).contiguous(), draft, None, acc, nxt, tgt)
    B.eh_check(ctx)
    clear = torch.from_numpy((full[3][4] >= P.NEAR_TIE).reshape(Bsz, 4)).to(DEV)
    assert torch.equal(tgt[clear], want[clear])
    sure = clear.all(dim=1)                                   # a near tie at the top may go either way
    assert int(sure.sum()) >= Bsz - 2
    stop = torch.where(torch.arange(Bsz, device=DEV) % 2 == 0, k, 1)
    assert torch.equal(acc[sure].long(), stop[sure])
    assert torch.equal(nxt[sure], want.gather(1, stop[:, None])[:, 0][sure])
    B.eh_destroy(ctx)


def _bias_heads(d, V, n_heads, rows, dtype, seed, kappa=0.6):
    w = G.Workload("biaslive", d=d, V=V, n_heads=n_heads, rows=rows, dtype=dtype, seed=seed, kappa=kappa)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    return w, heads, hid, [0.3 * torch.randn(V, generator=gen, device=DEV) for _ in range(n_heads)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_bias_heads_at_every_live_count(B, dtype):
    """The k-split kernel deals its grid out anew when less than half of a call's groups of 64 rows are
    live (here 7 groups: from 3 down); kernel and merge work the number of slices out on their own."""
    R = 400
    w, heads, hid, bs = _bias_heads(64, 9001, 1, R, dtype, 5)
    orc = _oracle(hid.h[0], heads.gamma[0], heads.beta[0], P.f64(heads.W[0]), bs[0], dtype == "bf16")
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=R, bias=bs)
    idx = torch.randperm(R, generator=torch.Generator().manual_seed(3)).to(torch.int32)
    for n in (0, 1, 64, 65, 128, 192, 193, 256, 257, 400):
        H, lse, am = _eval(B, ctx, 0, hid.h[0], R, row_idx=idx.to(DEV), n_rows_dev=torch.tensor([n], dtype=torch.int32, device=DEV))
        if n:
            P.compare_head(f"live{n}", H[:n], lse[:n], am[:n], tuple(x[idx[:n].numpy()] for x in orc), [])
        assert bool((H[n:] == 0).all()) and bool((lse[n:] == 0).all()) and bool((am[n:] == -7).all())
    B.eh_destroy(ctx)


def test_bias_cascade_whose_live_rows_fall_below_half(B):
    rows = 300
    w, heads, hid, bs = _bias_heads(96, 8200, 6, rows, "bf16", 8)
    full = [_oracle(hid.h[l], heads.gamma[l], heads.beta[l], P.f64(heads.W[l]), bs[l], True) for l in range(6)]
    full = [np.stack([f[i] for f in full]) for i in range(4)]
    tau = G.tau_for_schedule(full[0], 6)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows, bias=bs)
    ex, tok, H, nev = _ints(rows), _ints(rows), torch.zeros((6, rows), device=DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    B.eh_cascade(ctx, hid.h, rows, ex, tok, H, nev)
    torch.cuda.synchronize()
    P.compare_cascade("biasbelowhalf", ex, tok, H, full[0], full[2], full[3], tau, [])
    assert int(nev) == int((ex.long() + 1).sum())
    live = [int((ex >= l).sum()) for l in range(6)]
    assert live[0] > 256 and any(64 < n <= 128 for n in live) and live[-1] <= 128, live
    B.eh_destroy(ctx)


def test_few_live_rows_of_a_large_bias_call_have_the_whole_device(B):
    """40 live rows cost about the same whether the call was made for 40 rows or for 512 (1.1 times as
    much; 4 times when the grid followed the host's rows)."""
    w, heads, hid, bs = _bias_heads(1024, 50304, 1, 512, "bf16", 2)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=512, bias=bs)
    H, lse, am = torch.zeros(512, device=DEV), torch.zeros(512, device=DEV), _ints(512)
    n_dev = torch.tensor([40], dtype=torch.int32, device=DEV)

    def us(rows):
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                B.eh_eval(ctx, 0, hid.h[0], rows, H, lse, am, n_rows_dev=n_dev)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        return best

    us(512)
    assert us(512) < 2 * us(40)
    B.eh_destroy(ctx)


@pytest.mark.parametrize("rows", [67, 128, 129, 300])
def test_merge_of_four_and_sixteen_rows_a_workgroup(B, rows):
    """The merge of the partial statistics takes 4 rows a workgroup up to 128 rows and 16 beyond: both
    sides of the line, rows that fill neither, with and without the extra metrics, and the bits of
    one head at a time."""
    n_heads = 5
    w = G.Workload("merge", d=64, V=8203, n_heads=n_heads, rows=rows, dtype="bf16", seed=rows)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0] * n_heads, max_rows=rows)
    H, lse, p1, margin = (torch.zeros((n_heads, rows), device=DEV) for _ in range(4))
    am = _ints(n_heads, rows)
    B.eh_eval_heads_metrics(ctx, 0, n_heads, hid.h, rows, H, lse, am, p1, margin)
    for l in range(n_heads):
        orc = _oracle(hid.h[l], heads.gamma[l], heads.beta[l], P.f64(heads.W[l]), None, True)
        P.compare_head(f"merge{l}", H[l], lse[l], am[l], orc, [])
        pm_o, mg_o = O.head_metrics(P.f64(hid.h[l]), P.f64(heads.gamma[l]), P.f64(heads.beta[l]), P.f64(heads.W[l]), 1e-5, True)
        # exp of a difference of two logits of magnitude z: relative error that of their fp32 sums, 64 products deep
        np.testing.assert_allclose(P.f64(p1[l]), pm_o, rtol=2e-5)
        np.testing.assert_allclose(P.f64(margin[l]), mg_o, rtol=0, atol=2e-5)
    B.eh_eval_heads(ctx, 0, n_heads, hid.h, rows, H, lse, am)
    for l in range(n_heads):
        for a, b in zip(_eval(B, ctx, l, hid.h[l], rows), (H[l], lse[l], am[l])):
            assert torch.equal(a, b)
    B.eh_destroy(ctx)


@pytest.mark.parametrize("V", [49152, 49153, 57344, 57345])
@pytest.mark.parametrize("rows", [32, 33, 64])
def test_projection_of_33_to_64_rows_around_seven_tiles_a_pass(B, V, rows):
    """33 to 64 rows leave the k-split kernel where its passes have seven tiles (12 tiles of 16 rows a
    workgroup and more, up to 14): both sides of both lines."""
    w = G.Workload("seven", d=40, V=V, n_heads=2, rows=rows, dtype="bf16", seed=V + rows)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0, 0.0], max_rows=rows)
    H, lse, am = torch.zeros((2, rows), device=DEV), torch.zeros((2, rows), device=DEV), _ints(2, rows)
    B.eh_eval_heads(ctx, 0, 2, hid.h, rows, H, lse, am)
    for l in range(2):
        orc = _oracle(hid.h[l], heads.gamma[l], heads.beta[l], P.f64(heads.W[l]), None, True)
        P.compare_head(f"seven{l}", H[l], lse[l], am[l], orc, [])
        for a, b in zip(_eval(B, ctx, l, hid.h[l], rows), (H[l], lse[l], am[l])):
            assert torch.equal(a, b)
    B.eh_destroy(ctx)
