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


@pytest.mark.parametrize("rows", [65, 203, 256, 257])
def test_weights_past_the_caches(B, rows):
    """Several heads of more than 256 MB together: up to 256 rows their weights are read with non-temporal loads, of
    one head alone (or of 257 rows) with ordinary ones.  The same bits, with the extra metrics as well."""
    w = G.Workload("past", d=1024, V=50001, n_heads=3, rows=rows, dtype="bf16", seed=rows)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0] * 3, max_rows=rows)
    H, lse, am = torch.zeros((3, rows), device=DEV), torch.zeros((3, rows), device=DEV), _ints(3, rows)
    B.eh_eval_heads(ctx, 0, 3, hid.h, rows, H, lse, am)
    m = [torch.zeros((3, rows), device=DEV), torch.zeros((3, rows), device=DEV), _ints(3, rows)]
    prob, margin = torch.zeros((3, rows), device=DEV), torch.zeros((3, rows), device=DEV)
    B.eh_eval_heads_metrics(ctx, 0, 3, hid.h, rows, *m, prob, margin)
    for l in range(3):
        for a, b, c in zip(_eval(B, ctx, l, hid.h[l], rows), (H[l], lse[l], am[l]), (x[l] for x in m)):
            assert torch.equal(a, b) and torch.equal(a, c)
    assert bool((margin <= prob).all()) and bool((margin >= 0).all())
    B.eh_destroy(ctx)


@pytest.mark.parametrize("d,V,n,rows", [(1024, 50001, 4, 400), (1024, 50001, 4, 300), (512, 50001, 6, 230)])
def test_cascades_past_the_caches(B, d, V, n, rows):
    """Two launches per head on weights of more than 256 MB together, read with non-temporal loads, by rows that leave: two
    groups of live rows, one group of five and six blocks, then fewer."""
    w = G.Workload("pastcasc", d=d, V=V, n_heads=n, rows=rows, dtype="bf16", seed=rows + d, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    at = torch.arange(5, rows, 11, device=DEV)
    orc = [_oracle(hid.h[l][at], heads.gamma[l], heads.beta[l], P.f64(heads.W[l]), None, True) for l in range(n)]
    full = [np.stack([o[i] for o in orc]) for i in range(4)]
    tau = G.tau_for_schedule(full[0], n)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows)
    first = None
    for _ in range(3):
        ex, tok, H = _ints(rows), _ints(rows), torch.zeros((n, rows), device=DEV)
        B.eh_cascade(ctx, hid.h, rows, ex, tok, H, None)
        torch.cuda.synchronize()
        got = [ex, tok, H.view(torch.int32)]
        first = first or got
        assert all(torch.equal(a, b) for a, b in zip(got, first))
    print("live rows per head:", [int((ex >= l).sum()) for l in range(n)])
    P.compare_cascade("pastcasc", ex[at], tok[at], H[:, at], full[0], full[2], full[3], tau, [])
    B.eh_destroy(ctx)


@pytest.mark.parametrize("rows", [100, 180])
def test_verification_by_a_head_past_the_caches(B, rows):
    """A head of more than 256 MB by itself: the argmax-only projection reads it with non-temporal loads.  Targets by the oracle, on
    a row in seven, and by the entropy evaluation of the same rows on all."""
    d, V = 2560, 53001
    w = G.Workload("pastver", d=d, V=V, n_heads=1, rows=rows, dtype="bf16", seed=rows, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=rows)
    am = _eval(B, ctx, 0, hid.h[0], rows)[2]
    at = torch.arange(0, rows, 7, device=DEV)
    orc = _oracle(hid.h[0][at], heads.gamma[0], heads.beta[0], P.f64(heads.W[0]), None, True)
    for _ in range(2):
        acc, nxt, tgt = _ints(1), _ints(1), _ints(1, rows)
        B.dssd_verify(ctx, hid.h[0].reshape(1, rows, d).contiguous(), am[None, :-1].contiguous(), None, acc, nxt, tgt)
        assert torch.equal(tgt[0], am) and (int(acc), int(nxt)) == (rows - 1, int(am[-1]))
        clear = torch.from_numpy(orc[3] >= P.NEAR_TIE)
        assert bool(clear.any()) and torch.equal(tgt[0][at].cpu()[clear], torch.from_numpy(orc[2].astype(np.int32))[clear])
    B.eh_destroy(ctx)


@pytest.mark.parametrize("d,n,rows", [(1024, 3, 160), (768, 4, 192), (512, 2, 257), (768, 3, 320), (1024, 2, 353), (1536, 2, 384), (512, 2, 530)])
def test_five_and_six_blocks_on_weights_that_run_on(B, d, n, rows):
    """Groups of five and six blocks of rows with passes of several tiles, whose weights run on from pass to pass and head to
    head: one group past the caches (non-temporal loads), several groups (the shared form), with and without the
    extra metrics.  The oracle on a row of every block, and the bits of a head at a time, whose loads are ordinary ones."""
    w = G.Workload("runon", d=d, V=50001, n_heads=n, rows=rows, dtype="bf16", seed=rows + d)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0] * n, max_rows=rows)
    H, lse, am = torch.zeros((n, rows), device=DEV), torch.zeros((n, rows), device=DEV), _ints(n, rows)
    B.eh_eval_heads(ctx, 0, n, hid.h, rows, H, lse, am)
    m = [torch.zeros((n, rows), device=DEV), torch.zeros((n, rows), device=DEV), _ints(n, rows)]
    prob, margin = torch.zeros((n, rows), device=DEV), torch.zeros((n, rows), device=DEV)
    B.eh_eval_heads_metrics(ctx, 0, n, hid.h, rows, *m, prob, margin)
    at = torch.tensor(sorted(set(range(3, rows, 16)) | {rows - 1}), device=DEV)
    for l in range(n):
        orc = _oracle(hid.h[l][at], heads.gamma[l], heads.beta[l], P.f64(heads.W[l]), None, True)
        P.compare_head(f"runon{l}", H[l][at], lse[l][at], am[l][at], orc, [])
        y = O.layernorm(P.f64(hid.h[l][at]), P.f64(heads.gamma[l]), P.f64(heads.beta[l]), 1e-5, bf16_out=True)
        z = torch.from_numpy(y @ P.f64(heads.W[l]).T)
        p = torch.exp(torch.topk(z, 2, dim=1).values - torch.logsumexp(z, dim=1)[:, None])
        assert float((prob[l][at].double().cpu() - p[:, 0]).abs().max()) <= 2e-4
        assert float((margin[l][at].double().cpu() - (p[:, 0] - p[:, 1])).abs().max()) <= 2e-4
        for a, b, c in zip(_eval(B, ctx, l, hid.h[l], rows), (H[l], lse[l], am[l]), (x[l] for x in m)):
            assert torch.equal(a, b) and torch.equal(a, c)
    B.eh_destroy(ctx)


@pytest.mark.parametrize("V", [14999, 15000])
@pytest.mark.parametrize("Bsz,k", [(1, 16), (3, 6), (8, 7)])
def test_verification_on_both_sides_of_small_heads(B, V, Bsz, k):
    """Verifications of up to 64 positions: one launch below 6 * 10^6 elements of a head, three from there on.  Targets
    by the oracle; the accepted prefix ends at a planted mismatch in every second row."""
    d, rows = 400, Bsz * (k + 1)
    w = G.Workload("vline", d=d, V=V, n_heads=1, rows=rows, dtype="bf16", seed=rows, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    orc = _oracle(hid.h[0], heads.gamma[0], heads.beta[0], P.f64(heads.W[0]), None, True)
    want = torch.from_numpy(orc[2]).to(torch.int32).reshape(Bsz, k + 1).to(DEV)
    clear = torch.from_numpy(orc[3] >= P.NEAR_TIE).reshape(Bsz, k + 1).to(DEV)
    draft = want[:, :k].contiguous()
    draft[1::2, k // 2] = (draft[1::2, k // 2] + 1) % V
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=rows)
    for _ in range(2):
        acc, nxt, tgt = _ints(Bsz), _ints(Bsz), _ints(Bsz, k + 1)
        B.dssd_verify(ctx, hid.h[0].reshape(Bsz, k + 1, d).contiguous(), draft, None, acc, nxt, tgt)
        B.eh_check(ctx)
        assert torch.equal(tgt[clear], want[clear])
        for b in range(Bsz):
            if bool(clear[b].all()):
                stop = k // 2 if b % 2 else k
                assert (int(acc[b]), int(nxt[b])) == (stop, int(want[b, stop]))
    assert bool(clear.all(dim=1).any())
    B.eh_destroy(ctx)


@pytest.mark.parametrize("Bsz,k", [(2, 1), (40, 3), (30, 4), (9, 8), (1, 15), (1, 16), (3, 17), (1, 31), (1, 32), (1, 63), (2, 64), (1, 65), (2, 130), (1, 200)])
def test_verification_of_long_drafts(B, Bsz, k):
    """One, two and four positions a wave and prefixes that end on both sides of 64 positions and of 128, by a mismatch, by the draft's
    length or not at all.  Targets are the argmaxes of the same rows; the prefix rule by hand."""
    d, rows = 320, Bsz * (k + 1)
    w = G.Workload("long", d=d, V=20011, n_heads=1, rows=rows, dtype="bf16", seed=rows, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=rows)
    want = _eval(B, ctx, 0, hid.h[0], rows)[2].reshape(Bsz, k + 1)
    orc = _oracle(hid.h[0], heads.gamma[0], heads.beta[0], P.f64(heads.W[0]), None, True)
    clear = torch.from_numpy(orc[3] >= P.NEAR_TIE)
    assert torch.equal(want.reshape(-1).cpu()[clear], torch.from_numpy(orc[2].astype(np.int32))[clear])
    f = hid.h[0].reshape(Bsz, k + 1, d).contiguous()
    for stop in sorted({0, 1, k // 2, 62, 63, 64, 65, 127, 128, 129, k - 1, k} & set(range(k + 1))):
        for by_length in (False, True):
            draft, dlen = want[:, :k].clone(memory_format=torch.contiguous_format), None
            if by_length:
                dlen = torch.full((Bsz,), stop, dtype=torch.int32, device=DEV)
            elif stop < k:
                draft[:, stop] += 1
                draft[:, stop + 1:] = -1
            acc, nxt, tgt = _ints(Bsz), _ints(Bsz), _ints(Bsz, k + 1)
            B.dssd_verify(ctx, f, draft, dlen, acc, nxt, tgt)
            assert torch.equal(tgt, want) and bool((acc == stop).all()) and torch.equal(nxt, want[:, stop])
    B.eh_destroy(ctx)


@pytest.mark.parametrize("rows", [129, 160, 161, 192, 193, 300, 353])
@pytest.mark.parametrize("V", [3000, 20011, 40001, 50257, 60001])
def test_five_and_six_blocks_of_rows(B, rows, V):
    """Five and six blocks of 32 rows in a group (129 to 192 rows, and two groups of such).  In the two groups, of 300 and
    353 rows, four waves share the last blocks' tiles, one to four of the up to seven of a pass, and hand their statistics to one of
    them.  Passes of one to seven tiles, two passes a slice, and the second largest logit, which goes the same way."""
    w = G.Workload("five", d=104, V=V, n_heads=2, rows=rows, dtype="bf16", seed=V + rows)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0, 0.0], max_rows=rows)
    m = [torch.zeros((2, rows), device=DEV), torch.zeros((2, rows), device=DEV), _ints(2, rows)]
    prob, margin = torch.zeros((2, rows), device=DEV), torch.zeros((2, rows), device=DEV)
    B.eh_eval_heads_metrics(ctx, 0, 2, hid.h, rows, *m, prob, margin)
    acc, nxt, tgt = _ints(1), _ints(1), _ints(1, rows)
    B.dssd_verify(ctx, hid.h[1].reshape(1, rows, w.d).contiguous(), m[2][1][None, :-1].contiguous(), None, acc, nxt, tgt)
    for l in range(2):
        orc = _oracle(hid.h[l], heads.gamma[l], heads.beta[l], P.f64(heads.W[l]), None, True)
        P.compare_head(f"five{l}", m[0][l], m[1][l], m[2][l], orc, [])
        y = O.layernorm(P.f64(hid.h[l]), P.f64(heads.gamma[l]), P.f64(heads.beta[l]), 1e-5, bf16_out=True)
        z = torch.from_numpy(y @ P.f64(heads.W[l]).T)
        p = torch.exp(torch.topk(z, 2, dim=1).values - torch.logsumexp(z, dim=1)[:, None])
        assert float((prob[l].double().cpu() - p[:, 0]).abs().max()) <= 2e-4
        assert float((margin[l].double().cpu() - (p[:, 0] - p[:, 1])).abs().max()) <= 2e-4
        for a, b in zip(_eval(B, ctx, l, hid.h[l], rows), (m[0][l], m[1][l], m[2][l])):
            assert torch.equal(a, b)
    assert torch.equal(tgt[0], m[2][1]) and int(acc) == rows - 1 and int(nxt) == int(m[2][1][-1])
    B.eh_destroy(ctx)


@pytest.mark.parametrize("d,R", [(252, 33), (256, 33), (256, 64), (260, 65), (1024, 130)])
def test_fp32_heads_around_the_split_into_bf16_parts(B, d, R):
    """fp32 heads beyond 32 rows make their products of bf16 parts from d = 256 on."""
    w = G.Workload("f32split", d=d, V=9001, n_heads=2, rows=R, dtype="f32", seed=d + R, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    full = [_oracle(hid.h[l], heads.gamma[l], heads.beta[l], P.f64(heads.W[l]), None, False) for l in range(2)]
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [3.0, float("inf")], max_rows=R)
    for l in range(2):
        H, lse, am = _eval(B, ctx, l, hid.h[l], R)
        P.compare_head(f"f32split{l}", H, lse, am, full[l], [])
        # fp32 sums of d products, then of V exponentials: 2^-24 each, d / 32 and V / 512 in a row at most
        assert float((lse.double().cpu() - torch.from_numpy(full[l][1])).abs().max()) <= 2.0 ** -24 * (d / 32 + 9001 / 512) * 16
    ex, tok, H = _ints(R), _ints(R), torch.zeros((2, R), device=DEV)
    B.eh_cascade(ctx, hid.h, R, ex, tok, H, None)
    torch.cuda.synchronize()
    full = [np.stack([f[i] for f in full]) for i in range(4)]
    P.compare_cascade("f32split", ex, tok, H, full[0], full[2], full[3], [3.0, float("inf")], [])
    B.eh_destroy(ctx)


@pytest.mark.parametrize("exponent", [-90, -60, -20, 0, 12])
def test_fp32_products_keep_their_24_bits(B, exponent):
    """One word and one weight that is not zero: the log-sum-exp is the product itself.  Three bf16 parts hold a fp32
    value exactly, and the products left out are below 2^-22 of it (the LayerNorm output, rounded to fp32, adds 2^-24).  Up
    to 2^12: the statistics take 2^(z log2 e - m), whose exponent a logit above 2^20 no longer gives to a fraction of one."""
    d, R = 256, 40
    g = torch.Generator().manual_seed(exponent + 100)
    h = torch.randn((R, d), generator=g)
    for at in (0, 7, 100, 255):
        W = torch.zeros((1, d))
        W[0, at] = (1.0 + float(torch.rand(1, generator=g))) * 2.0 ** exponent
        ctx = B.eh_create([W.to(DEV)], [torch.ones(d, device=DEV)], [torch.zeros(d, device=DEV)], [0.0], max_rows=R)
        H, lse, am = _eval(B, ctx, 0, h.to(DEV), R)
        B.eh_destroy(ctx)
        z = O.layernorm(P.f64(h), np.ones(d), np.zeros(d), 1e-5, bf16_out=False)[:, at] * float(W[0, at])
        assert np.abs(lse.double().cpu().numpy() / z - 1.0).max() <= 2.0 ** -21 and bool((am == 0).all())


def _check_bias_heads(B, d, V, rows):
    w, heads, hid, bs = _bias_heads(d, V, 2, rows, "bf16", V + rows)
    bs[1] *= 20.0
    orc = [_oracle(hid.h[l], heads.gamma[l], heads.beta[l], P.f64(heads.W[l]), bs[l], True) for l in range(2)]
    tau = [float(np.median(orc[0][0])), float("inf")]
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows, bias=bs)
    for l in range(2):
        P.compare_head(f"bias{l}", *_eval(B, ctx, l, hid.h[l], rows), orc[l], [])
    full = [np.stack([o[i] for o in orc]) for i in range(4)]
    ex, tok, H = _ints(rows), _ints(rows), torch.zeros((2, rows), device=DEV)
    B.eh_cascade(ctx, hid.h, rows, ex, tok, H, None)
    torch.cuda.synchronize()
    P.compare_cascade("biasbatched", ex, tok, H, full[0], full[2], full[3], tau, [])
    acc, nxt, tgt = _ints(1), _ints(1), _ints(1, rows)
    B.dssd_verify(ctx, hid.h[1].reshape(1, rows, w.d).contiguous(), torch.from_numpy(orc[1][2][None, :-1].astype(np.int32)).to(DEV), None, acc, nxt, tgt)
    clear = torch.from_numpy(orc[1][3] >= P.NEAR_TIE)
    assert torch.equal(tgt[0].cpu()[clear], torch.from_numpy(orc[1][2].astype(np.int32))[clear])
    B.eh_destroy(ctx)


@pytest.mark.parametrize("V,rows", [(50257, 33), (50257, 64), (1500, 65), (9001, 129), (20011, 160), (40001, 200), (60001, 300), (17, 513)])
def test_batched_kernel_with_a_bias_vector(B, V, rows):
    """bf16 heads with a bias vector beyond 32 rows (64 where a pass has fewer than seven tiles): the bias is added to
    the finished sums.  Ragged last tiles, a bias that decides the argmax, a cascade, and a verification."""
    _check_bias_heads(B, 136, V, rows)


@pytest.mark.parametrize("d,V,rows", [
    (136, 8192, 128), (136, 8193, 128), (136, 8192, 129), (136, 8192, 256), (136, 8192, 257), (136, 4096, 512), (136, 4096, 513),
    (136, 2720, 190), (136, 2721, 190), (136, 16, 321), (3072, 50304, 33), (3064, 50304, 33), (3072, 49153, 64), (3072, 50304, 65)])
def test_bias_heads_on_both_sides_of_their_lines(B, d, V, rows):
    """Heads with a bias vector on few words for their rows, and of long k loops on up to 64 rows, run on the k-split kernel:
    each line from both sides."""
    _check_bias_heads(B, d, V, rows)


@pytest.mark.parametrize("dtype,d,V,rows", [
    ("bf16", 1536, 9001, 9), ("bf16", 1536, 9001, 20), ("bf16", 1536, 9001, 64), ("bf16", 1536, 9001, 65), ("bf16", 1536, 50257, 64),
    ("bf16", 1536, 20011, 300), ("f32", 1024, 9001, 40), ("f32", 1024, 9001, 130)])
def test_bias_vectors_with_an_offset(B, dtype, d, V, rows):
    """A bias vector may have any common offset: it is added to finished sums.  At 10^4 a logit is then rounded to 2^-11,
    once, and the entropy follows with the mean of |log p + H|, of size 1 (H + 2^-11 and 2^-10); a sum that starts from the bias
    is rounded d / 16 times."""
    w, heads, hid, bs = _bias_heads(d, V, 1, rows, dtype, V + rows, kappa=0.2)
    bs[0] += 1e4
    orc = _oracle(hid.h[0], heads.gamma[0], heads.beta[0], P.f64(heads.W[0]), bs[0], dtype == "bf16")
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=rows, bias=bs)
    H, lse, am = _eval(B, ctx, 0, hid.h[0], rows)
    B.eh_destroy(ctx)
    print("entropies off by", float((H.double().cpu() - torch.from_numpy(orc[0])).abs().max()))
    P.compare_head("offset", H, lse, am, orc, [])


@pytest.mark.parametrize("d", [512, 776, 2048])
def test_bias_heads_keep_their_precision_beyond_the_few_rows(B, d):
    """The sums of a head with a bias vector are made of quarters of k on both sides of the line between the kernels: the rows 32
    at a time (the k-split kernel) and all at once (the batched one) are equally far from 64 bits.  (Norms of 320 errors, by
    chance within 1.25 of each other; one chain over k has log-sum-exps more than twice as far.)"""
    rows = 320
    w, heads, hid, bs = _bias_heads(d, 20011, 1, rows, "bf16", d, kappa=1.0)
    orc = _oracle(hid.h[0], heads.gamma[0], heads.beta[0], P.f64(heads.W[0]), bs[0], True)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=rows, bias=bs)
    few = [_eval(B, ctx, 0, hid.h[0][i:i + 32].contiguous(), 32) for i in range(0, rows, 32)]
    off = [[float(np.linalg.norm(x.double().cpu().numpy() - o)) for x, o in zip(got, orc)] for got in
           ([torch.cat([f[i] for f in few]) for i in range(2)], _eval(B, ctx, 0, hid.h[0], rows)[:2])]
    print("errors of entropies and log-sum-exps, 32 rows at a time and all at once:", off)
    assert off[1][0] <= 1.5 * off[0][0] and off[1][1] <= 1.5 * off[0][1]
    B.eh_destroy(ctx)


@pytest.mark.parametrize("dtype,d,V,rows", [
    ("bf16", 136, 9001, 9), ("bf16", 136, 9001, 33), ("bf16", 136, 9001, 64), ("bf16", 136, 50257, 64), ("bf16", 136, 9001, 65),
    ("bf16", 136, 20011, 160), ("f32", 136, 9001, 40), ("f32", 256, 9001, 40), ("f32", 256, 9001, 70)])
@pytest.mark.parametrize("mask", [-np.inf, -3.4028234663852886e38, -1e30])
def test_bias_vectors_that_mask_words(B, dtype, d, V, rows, mask):
    """A bias of -infinity, of the lowest float or of a very low one takes a word out: the statistics are those of the
    words that are left, also where whole tiles and a whole slice of the vocabulary are masked."""
    w, heads, hid, bs = _bias_heads(d, V, 1, rows, dtype, V + rows)
    out = torch.zeros(V, dtype=torch.bool, device=DEV)
    out[::3] = True
    out[256:1024] = True
    out[-40:] = True
    bs[0][out] = mask
    low = bs[0].clone()
    low[out] = -1e6  # a probability of 0 in 64 bits as well
    orc = _oracle(hid.h[0], heads.gamma[0], heads.beta[0], P.f64(heads.W[0]), low, dtype == "bf16")
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=rows, bias=bs)
    P.compare_head("masked", *_eval(B, ctx, 0, hid.h[0], rows), orc, [])
    B.eh_destroy(ctx)


@pytest.mark.parametrize("dtype,d,V,rows", [
    ("bf16", 136, 9001, 9), ("bf16", 136, 9001, 33), ("bf16", 136, 9001, 64), ("bf16", 136, 50257, 64), ("bf16", 136, 9001, 65),
    ("bf16", 136, 20011, 160), ("f32", 136, 9001, 40), ("f32", 256, 9001, 40)])
@pytest.mark.parametrize("top,rest", [(1.6e7, 0.0), (1e9, 0.0), (1e14, 0.0), (1e30, 0.0), (3.4028234663852886e38, 0.0), (-1e30, -2e30)])
def test_bias_vectors_that_force_a_word(B, dtype, d, V, rows, top, rest):
    """A bias far above all others forces a word, however far: the argmax, a verification's targets and a cascade's
    tokens.  Up to 10^9 the entropy (0) and the log-sum-exp as well; beyond, a product z log2 e is rounded by more than an
    exponent holds."""
    w, heads, hid, bs = _bias_heads(d, V, 2, rows, dtype, V + rows)
    word = V // 3
    for b in bs:
        b += rest
        b[word] = top
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0, 0.0], max_rows=rows, bias=bs)
    for l in range(2):
        H, lse, am = _eval(B, ctx, l, hid.h[l], rows)
        assert bool((am == word).all())
        if abs(top) <= 1e9:
            assert float(H.abs().max()) <= P.TOL_H and float((lse / top - 1.0).abs().max()) <= P.TOL_LSE_REL
    ex, tok, H = _ints(rows), _ints(rows), torch.zeros((2, rows), device=DEV)
    B.eh_cascade(ctx, hid.h, rows, ex, tok, H, None)
    assert bool((tok == word).all())
    acc, nxt, tgt = _ints(1), _ints(1), _ints(1, rows)
    B.dssd_verify(ctx, hid.h[1].reshape(1, rows, w.d).contiguous(), torch.full((1, rows - 1), word, dtype=torch.int32, device=DEV), None, acc, nxt, tgt)
    assert bool((tgt == word).all()) and (int(acc), int(nxt)) == (rows - 1, word)
    B.eh_destroy(ctx)


def _heads_with_a_switch(d, V, n_heads, rows, dtype, seed):
    """Heads whose LayerNorm output is 1 at the last place in every row, where all words have weight 0."""
    w = G.Workload("switch", d=d, V=V, n_heads=n_heads, rows=rows, dtype=dtype, seed=seed, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    for W, g, b in zip(heads.W, heads.gamma, heads.beta):
        W[:, -1] = 0.0
        g[-1] = 0.0
        b[-1] = 1.0
    return heads, hid


@pytest.mark.parametrize("dtype,d,V,rows,bias", [
    ("bf16", 256, 9001, 20, False), ("bf16", 256, 9001, 33, False), ("bf16", 256, 9001, 64, False), ("bf16", 256, 9001, 64, True),
    ("bf16", 256, 9001, 65, True), ("bf16", 256, 20011, 160, True), ("f32", 128, 9001, 20, False), ("f32", 256, 9001, 32, False),
    ("f32", 256, 9001, 40, True), ("f32", 128, 9001, 130, True)])
def test_weights_of_infinity_that_mask_words(B, dtype, d, V, rows, bias):
    """A weight of -infinity on a place of the LayerNorm output that is 1 in every row takes its word out: the
    statistics are those of the words that are left, also where whole tiles are masked; in a cascade as well.  (d such that
    the four waves of the k-split kernel have an even number of k-steps each: none runs one on activations of 0.)"""
    heads, hid = _heads_with_a_switch(d, V, 2, rows, dtype, V + rows)
    gen = torch.Generator(device=DEV).manual_seed(rows)
    bs = [0.3 * torch.randn(V, generator=gen, device=DEV) for _ in range(2)] if bias else None
    out = torch.zeros(V, dtype=torch.bool, device=DEV)
    out[::3] = True
    out[256:1024] = True
    out[-40:] = True
    low = torch.where(out, -1e6, 0.0)  # a probability of 0 in 64 bits as well
    orc = [_oracle(hid.h[l], heads.gamma[l], heads.beta[l], P.f64(heads.W[l]), low + bs[l] if bias else low, dtype == "bf16") for l in range(2)]
    for W in heads.W:
        W[out, -1] = -np.inf
    tau = [float(np.median(orc[0][0])), float("inf")]
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows, bias=bs)
    for l in range(2):
        P.compare_head(f"switch{l}", *_eval(B, ctx, l, hid.h[l], rows), orc[l], [])
    ex, tok, H = _ints(rows), _ints(rows), torch.zeros((2, rows), device=DEV)
    B.eh_cascade(ctx, hid.h, rows, ex, tok, H, None)
    torch.cuda.synchronize()
    full = [np.stack([o[i] for o in orc]) for i in range(4)]
    P.compare_cascade("switch", ex, tok, H, full[0], full[2], full[3], tau, [])
    B.eh_destroy(ctx)


@pytest.mark.parametrize("d,rows,bias", [(128, 20, False), (256, 32, False), (256, 40, False), (128, 40, True), (256, 130, True)])
def test_fp32_weights_of_infinity_that_force_a_word(B, d, rows, bias):
    """A weight of infinity does not split into bf16 parts: its word has the largest logit all the same."""
    heads, hid = _heads_with_a_switch(d, 9001, 1, rows, "f32", rows)
    heads.W[0][4321, -1] = np.inf
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=rows, bias=[torch.zeros(9001, device=DEV)] if bias else None)
    H, lse, am = _eval(B, ctx, 0, hid.h[0], rows)
    assert bool((am == 4321).all())
    acc, nxt, tgt = _ints(1), _ints(1), _ints(1, rows)
    B.dssd_verify(ctx, hid.h[0].reshape(1, rows, d).contiguous(), torch.full((1, rows - 1), 4321, dtype=torch.int32, device=DEV), None, acc, nxt, tgt)
    assert bool((tgt == 4321).all()) and (int(acc), int(nxt)) == (rows - 1, 4321)
    B.eh_destroy(ctx)


@pytest.mark.parametrize("R,counts", [(192, (129, 150, 170, 192)), (400, (288, 300, 340, 384))])
def test_rows_do_not_depend_on_their_place_in_the_list(B, R, counts):
    """A live count on the device comes with a list of rows whose order is that of their arrival: the bits of a row are
    the same at every place, with five or six blocks of 32 in a group and several tiles a slice, too."""
    w = G.Workload("place", d=160, V=40001, n_heads=1, rows=R, dtype="bf16", seed=R)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=R)
    gen = torch.Generator().manual_seed(R)
    for n in counts:
        live = torch.tensor([n], dtype=torch.int32, device=DEV)
        one = _eval(B, ctx, 0, hid.h[0], R, n_rows_dev=live)
        for _ in range(2):
            p = torch.randperm(n, generator=gen)
            other = _eval(B, ctx, 0, hid.h[0], R, row_idx=torch.cat([p, torch.arange(n, R)]).to(torch.int32).to(DEV), n_rows_dev=live)
            for a, b in zip(other, one):
                assert torch.equal(a[:n], b[:n][p.to(DEV)])
    B.eh_destroy(ctx)


@pytest.mark.parametrize("dtype,d,V,R,counts", [("bf16", 136, 8001, 128, (33, 65, 90, 128)), ("bf16", 136, 20011, 200, (65, 150, 192)),
                                                ("f32", 256, 20011, 200, (33, 65, 100, 161)), ("f32", 128, 20011, 100, (33, 65, 90))])
def test_rows_of_bias_and_fp32_heads_do_not_depend_on_their_place(B, dtype, d, V, R, counts):
    """The same for heads with a bias vector and fp32 heads with one, on the k-split kernel and the batched one: a group's last
    block of rows alone or beside another, and lists of every number of groups."""
    w, heads, hid, bs = _bias_heads(d, V, 1, R, dtype, V + R)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=R, bias=bs)
    gen = torch.Generator().manual_seed(R)
    for n in counts:
        live = torch.tensor([n], dtype=torch.int32, device=DEV)
        one = _eval(B, ctx, 0, hid.h[0], R, n_rows_dev=live)
        p = torch.randperm(n, generator=gen)
        other = _eval(B, ctx, 0, hid.h[0], R, row_idx=torch.cat([p, torch.arange(n, R)]).to(torch.int32).to(DEV), n_rows_dev=live)
        for a, b in zip(other, one):
            assert torch.equal(a[:n], b[:n][p.to(DEV)])
    B.eh_destroy(ctx)


@pytest.mark.parametrize("rows", [192, 230, 400])
def test_cascades_of_two_launches_repeat_to_the_bit(B, rows):
    """V and the live counts are such that groups of five and six blocks of rows with several tiles a slice come up."""
    n = 8
    w = G.Workload("again", d=160, V=40001, n_heads=n, rows=rows, dtype="bf16", seed=rows, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    full = P.oracle_all_heads(heads, hid.h, True, rows=slice(0, 32))
    tau = G.tau_for_schedule(full[0], n)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows)
    first = None
    for _ in range(8):
        ex, tok, H = _ints(rows), _ints(rows), torch.zeros((n, rows), device=DEV)
        B.eh_cascade(ctx, hid.h, rows, ex, tok, H, None)
        torch.cuda.synchronize()
        got = [ex, tok, H.view(torch.int32)]
        first = first or got
        assert all(torch.equal(a, b) for a, b in zip(got, first))
    live = [int((ex >= l).sum()) for l in range(1, n)]
    assert any(128 < x <= 192 or 256 < x <= 384 for x in live), live
    P.compare_cascade("again", ex[:32], tok[:32], H[:, :32], full[0], full[2], full[3], tau, [])
    B.eh_destroy(ctx)
