"""Edge cases of the method on every kernel path, through the C ABI, against the oracle:
exact ties at the top (lowest index wins, eq. (2) with the build's tie rule), entropies exactly
on a threshold and beside it (strict H < tau, Sections 3.4.2 and 4.3.1), heads that start with
no live row, rows with NaN / Inf hidden states, the persistent kernel's give-up path, and the
calibration level met exactly (Section 3.4.1).

Row counts pick the kernel: at most 16 rows run the decode kernel, more the batched ones (up to 64
rows, and heads with a bias vector at any number, the k-split projection; beyond, bf16 in 32-row
blocks, one per wave, fp32 in 16-row blocks).  Cascades of bf16 heads of 17 to
26 + V (d + 620) / 10^6 rows (at least 64; 64 where heads are small) and verifications of up to 64 positions run
in one persistent launch.
"""
import math

import numpy as np
import pytest
import torch

from oracle import eh_oracle as O
from workloads import generators as G
from tests import parity_util as P

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
V_BIG = G.V_PYTHIA

# (lower, higher) vocabulary rows that are made to tie at the top, one pair per head.  With 256
# workgroups over 50304 rows a slice is 196.5 rows: the pairs sit in one 16-row tile, in one
# slice but different tiles, on both sides of the first slice boundary inside a tile (row 196
# cuts tile 12), in neighbouring slices and at the two ends of the vocabulary.
PAIRS_BIG = [(1000, 1003), (1010, 1100), (194, 198), (150, 250), (5, 50000), (50287, 50303)]


@pytest.fixture(scope="module")
def B():
    from paper_2407_21082_amd import binding
    return binding


def _outs(n):
    return (torch.full((n,), float("nan"), device=DEV), torch.full((n,), float("nan"), device=DEV),
            torch.full((n,), -7, dtype=torch.int32, device=DEV))


def _plant_ties(w, heads, hid, pairs, bf16, value=256.0):
    """Head l gets two identical vocabulary rows pairs[l] whose only non-zero weight is `value`
    at a hidden index where the LayerNorm output of most rows is clearly positive: their logit
    value * y_j is a single exact product on either side (no rounding, whatever the order of
    summation), equal for the two rows, and for those rows the largest by far."""
    wins = []
    for l, (a, b) in enumerate(pairs):
        y = O.layernorm(P.f64(hid.h[l]), P.f64(heads.gamma[l]), P.f64(heads.beta[l]), w.ln_eps, bf16_out=bf16)
        ok = y > 0.2
        j0 = int(np.argmax(ok.sum(axis=0) + 1000 * ok[0]))          # row 0 must be among them
        assert ok[0, j0] and ok[:, j0].sum() >= max(1, y.shape[0] // 4)
        heads.W[l][a].zero_()
        heads.W[l][a, j0] = value
        heads.W[l][b] = heads.W[l][a]
        wins.append(np.flatnonzero(ok[:, j0]))
    return wins


def _check_tie_head(name, got, orc, rows_tied, pair):
    """Statistics within tolerance everywhere, and on the rows where the oracle sees an exact
    tie of the planted pair at the top the index is the lower one -- no near-tie excuse."""
    H, lse, am = got
    H_o, lse_o, am_o, gap_o = orc
    P.compare_head(name, H, lse, am, orc, [])
    am = am.cpu().numpy()
    tied = [r for r in rows_tied if gap_o[r] == 0.0 and am_o[r] == pair[0]]
    assert len(tied) >= 1, f"{name}: the planted pair wins nowhere"
    for r in tied:
        assert am[r] == pair[0], f"{name}: row {r} picked {am[r]}, the tie {pair} goes to the lower index"
    return len(tied)


# ------------------------------------------------------------------ ties: eh_eval on every path
@pytest.mark.parametrize("dtype,d,rows", [("bf16", 1024, 16), ("bf16", 1024, 1), ("bf16", 256, 40), ("bf16", 256, 150),
                                          ("f32", 512, 16), ("f32", 512, 32)])
def test_exact_tie_at_the_top_goes_to_the_lower_index(B, dtype, d, rows):
    bf16 = dtype == "bf16"
    w = G.Workload("tie", d=d, V=V_BIG, n_heads=len(PAIRS_BIG), rows=rows, dtype=dtype, seed=700 + d + rows)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    wins = _plant_ties(w, heads, hid, PAIRS_BIG, bf16)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, G.tau_linear(w), max_rows=rows)
    total = 0
    for l, pair in enumerate(PAIRS_BIG):
        H, lse, am = _outs(rows)
        B.eh_eval(ctx, l, hid.h[l], rows, H, lse, am)
        torch.cuda.synchronize()
        orc = P.oracle_head(hid.h[l], heads.gamma[l], heads.beta[l], heads.W[l], bf16)
        total += _check_tie_head(f"tie/{dtype}/{rows}/head{l}", (H, lse, am), orc, wins[l], pair)
    B.eh_check(ctx)
    B.eh_destroy(ctx)
    assert total >= len(PAIRS_BIG)


@pytest.mark.parametrize("rows", [9, 40])
def test_exact_tie_with_a_bias_vector(B, rows):
    pairs = [(100, 103), (7, 5100), (2047, 2049)]
    w = G.Workload("tiebias", d=128, V=5200, n_heads=len(pairs), rows=rows, dtype="bf16", seed=31 + rows)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    wins = _plant_ties(w, heads, hid, pairs, True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(9)
    bias = [torch.randn(w.V, generator=gen, device=DEV) for _ in pairs]
    for l, (a, b) in enumerate(pairs):
        bias[l][b] = bias[l][a]
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, G.tau_linear(w), max_rows=rows, bias=bias)
    for l, pair in enumerate(pairs):
        H, lse, am = _outs(rows)
        B.eh_eval(ctx, l, hid.h[l], rows, H, lse, am)
        torch.cuda.synchronize()
        orc = O.head_eval(P.f64(hid.h[l]), P.f64(heads.gamma[l]), P.f64(heads.beta[l]), P.f64(heads.W[l]), 1e-5, True,
                          bias=P.f64(bias[l]))
        _check_tie_head(f"tiebias/{rows}/head{l}", (H, lse, am), orc, wins[l], pair)
    B.eh_destroy(ctx)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Bsz,k", [(3, 3), (5, 4), (16, 8)])
def test_exact_tie_in_the_verification_targets(B, dtype, Bsz, k):
    """dssd_verify with ties at the top of the model's head: 12 positions (three launches, the
    k-split projection), 25 (bf16: one persistent launch) and 144 (three launches, the batched projection)."""
    bf16 = dtype == "bf16"
    rows = Bsz * (k + 1)
    pair = (1200, 30000)
    w = G.Workload("tiever", d=256, V=V_BIG, n_heads=1, rows=rows, dtype=dtype, seed=11 * Bsz + k)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV, amp=torch.full((rows,), 1.5))    # every other row decides clearly
    _plant_ties(w, heads, hid, [pair], bf16)
    f_final = hid.h[0].reshape(Bsz, k + 1, w.d).contiguous()
    f64 = P.f64
    _, _, tgt_o, gap_o = O.dssd_verify(f64(f_final), np.zeros((Bsz, k), dtype=np.int64), f64(heads.gamma[0]),
                                       f64(heads.beta[0]), f64(heads.W[0]), None, 1e-5, bf16)
    # drafts: the model's own targets with every fifth one changed, so prefixes of all lengths occur
    draft = tgt_o[:, :k].copy()
    flat = draft.reshape(-1)
    flat[2::5] = (flat[2::5] + 1) % w.V
    acc_o, nxt_o, tgt_o, gap_o = O.dssd_verify(f64(f_final), draft, f64(heads.gamma[0]), f64(heads.beta[0]),
                                               f64(heads.W[0]), None, 1e-5, bf16)
    tied = np.flatnonzero((gap_o.reshape(-1) == 0.0) & (tgt_o.reshape(-1) == pair[0]))
    assert len(tied) >= 1
    assert (np.delete(gap_o.reshape(-1), tied) > 1e-3).all()
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [float("inf")], max_rows=rows)
    acc = torch.full((Bsz,), -1, dtype=torch.int32, device=DEV)
    nxt = torch.full((Bsz,), -1, dtype=torch.int32, device=DEV)
    tgt = torch.full((Bsz, k + 1), -1, dtype=torch.int32, device=DEV)
    B.dssd_verify(ctx, f_final, torch.from_numpy(draft).to(torch.int32).to(DEV).contiguous(), None, acc, nxt, tgt)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(tgt.cpu().numpy(), tgt_o)
    np.testing.assert_array_equal(acc.cpu().numpy(), acc_o)
    np.testing.assert_array_equal(nxt.cpu().numpy(), nxt_o)
    B.eh_destroy(ctx)


# ------------------------------------------------------------------ the exit test at the threshold
def _f32(x):
    return float(np.float32(x))


def test_exit_decide_on_exact_boundary_entropies(B):
    """eh_exit_decide takes the entropies from the caller, so values on the threshold, one unit in
    the last place beside it, NaN, the infinities and the two zeros can be fed exactly; the rule is
    the oracle's exit_rule (strict H < tau; the last head always answers)."""
    taus = [1.5, 0.0, float("-inf"), float("inf"), 0.25]
    w = G.Workload("decide", d=64, V=64, n_heads=len(taus), rows=4, dtype="bf16", seed=3)
    heads = G.make_heads(w, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, taus, max_rows=400)
    up = lambda x: _f32(np.nextafter(np.float32(x), np.float32(np.inf)))
    dn = lambda x: _f32(np.nextafter(np.float32(x), np.float32(-np.inf)))
    vals = [1.5, up(1.5), dn(1.5), 0.0, -0.0, up(0.0), dn(0.0), float("nan"), float("inf"), float("-inf"),
            0.25, up(0.25), dn(0.25), 3.0e38, -3.0e38, 1e-45, -1e-45, 0.7, 2.0, -1.0]
    rng = np.random.default_rng(5)
    Hh = np.array(vals * 15, dtype=np.float32)             # 300 positions: more than one sweep of the workgroup
    rng.shuffle(Hh)
    n = len(Hh)
    H = torch.from_numpy(Hh).to(DEV)
    am = torch.arange(1000, 1000 + n, dtype=torch.int32, device=DEV)
    perm = torch.from_numpy(rng.permutation(n).astype(np.int32)).to(DEV)
    for head in range(len(taus)):
        for idx, n_dev in ((None, None), (perm, None), (perm, 173), (None, 0)):
            ex = torch.full((n,), -1, dtype=torch.int32, device=DEV)
            tok = torch.full((n,), -1, dtype=torch.int32, device=DEV)
            act = torch.full((n,), -9, dtype=torch.int32, device=DEV)
            cnt = torch.full((1,), -9, dtype=torch.int32, device=DEV)
            nd = None if n_dev is None else torch.tensor([n_dev], dtype=torch.int32, device=DEV)
            B.eh_exit_decide(ctx, head, H, am, n, ex, tok, act, cnt, row_idx=idx, n_rows_dev=nd)
            torch.cuda.synchronize()
            live = n if n_dev is None else n_dev
            want_ex = np.full(n, -1)
            want_tok = np.full(n, -1)
            stay = []
            for p in range(live):
                r = p if idx is None else int(perm[p])
                # the oracle's rule on a two-head stack: this head, then one that always answers
                leaves = head == len(taus) - 1 or O.exit_rule([float(Hh[p]), 0.0], [taus[head], math.inf]) == 0
                if leaves:
                    want_ex[r], want_tok[r] = head, 1000 + p
                else:
                    stay.append(r)
            np.testing.assert_array_equal(ex.cpu().numpy(), want_ex)
            np.testing.assert_array_equal(tok.cpu().numpy(), want_tok)
            assert int(cnt.item()) == len(stay) and act[:len(stay)].tolist() == stay, (head, n_dev)
    B.eh_destroy(ctx)


@pytest.mark.parametrize("dtype,rows", [("bf16", 8), ("bf16", 40), ("bf16", 150), ("f32", 12), ("f32", 40)])
def test_cascade_is_strict_at_its_own_entropy(B, dtype, rows):
    """The exit test inside the cascade kernels (persistent kernel; cascade step kernel behind the
    batched ones): the threshold of head 0 is set to the very float the library reports as a row's
    entropy, and to its two neighbours.  Equal or below: the row goes on; one unit above: it leaves."""
    w = G.Workload("strict", d=256, V=3000, n_heads=3, rows=rows, dtype=dtype, seed=rows + 40)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    # the library's own entropies of every head on every row: a cascade in which no exit head ever
    # fires reports them all (the same kernels, hence the same floats, as the cascades below)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [float("-inf"), float("-inf"), 0.0], max_rows=rows)
    Hg = torch.zeros((3, rows), device=DEV)
    Ag = torch.zeros((3, rows), dtype=torch.int32, device=DEV)
    ex0 = torch.full((rows,), -1, dtype=torch.int32, device=DEV)
    tok0 = torch.full((rows,), -1, dtype=torch.int32, device=DEV)
    B.eh_cascade(ctx, hid.h, rows, ex0, tok0, Hg, None)
    for l in range(3):
        B.eh_eval(ctx, l, hid.h[l], rows, None, None, Ag[l])
    torch.cuda.synchronize()
    assert (ex0 == 2).all() and torch.equal(tok0, Ag[2]) and torch.isfinite(Hg).all()
    B.eh_destroy(ctx)
    Hn, An = Hg.cpu().numpy(), Ag.cpu().numpy()
    r_star = int(np.argsort(Hn[0])[rows // 2])              # a row in the middle of head 0's entropies
    h0 = np.float32(Hn[0, r_star])
    for tau0, leaves in ((h0, False), (np.nextafter(h0, np.float32(-np.inf)), False),
                         (np.nextafter(h0, np.float32(np.inf)), True)):
        tau = [float(tau0), float("-inf"), float("inf")]
        ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows)
        ex = torch.full((rows,), -1, dtype=torch.int32, device=DEV)
        tok = torch.full((rows,), -1, dtype=torch.int32, device=DEV)
        Hout = torch.zeros((3, rows), device=DEV)
        nev = torch.zeros(1, dtype=torch.int64, device=DEV)
        B.eh_cascade(ctx, hid.h, rows, ex, tok, Hout, nev)
        torch.cuda.synchronize()
        B.eh_check(ctx)
        B.eh_destroy(ctx)
        want = np.array([O.exit_rule([float(Hn[l, r]) for l in range(3)], tau) for r in range(rows)])
        np.testing.assert_array_equal(ex.cpu().numpy(), want)
        assert (want[r_star] == 0) == leaves
        np.testing.assert_array_equal(tok.cpu().numpy(), An[want, np.arange(rows)])
        Ho = Hout.cpu().numpy()
        # head 0 sees the same columns in both cascades: the same floats.  Later heads see the
        # survivors compacted, and a different number of token blocks per wave may round the last bit
        # differently; beyond the exit nothing is evaluated.
        assert (Ho[0] == Hn[0]).all()
        for r in range(rows):
            assert np.allclose(Ho[1:want[r] + 1, r], Hn[1:want[r] + 1, r], rtol=2e-6, atol=2e-6)
            assert np.isnan(Ho[want[r] + 1:, r]).all()
        assert int(nev.item()) == int((want + 1).sum())


# ------------------------------------------------------------------ heads that start with no live row
@pytest.mark.parametrize("dtype,rows", [("bf16", 70), ("bf16", 150), ("bf16", 12), ("f32", 40)])
def test_cascade_with_heads_that_have_no_live_row(B, dtype, rows):
    bf16 = dtype == "bf16"
    w = G.Workload("empty", d=128, V=2000, n_heads=5, rows=rows, dtype=dtype, seed=rows + 5, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    full = P.oracle_all_heads(heads, hid.h, bf16)
    srt = np.sort(full[0][0])
    i = max(range(rows // 3, 2 * rows // 3), key=lambda j: srt[j] - srt[j - 1])    # the widest gap near the middle
    med = float(srt[i] + srt[i - 1]) / 2
    assert np.abs(full[0][0] - med).min() > 2e-3
    f64 = P.f64
    for name, tau in (("all leave at head 0", [float("inf")] * 5),
                      ("half at head 0, the rest at head 2", [med, float("-inf"), float("inf"), 1.0, float("inf")])):
        ref = O.cascade([f64(hid.h[l]) for l in range(5)], [f64(g) for g in heads.gamma], [f64(b) for b in heads.beta],
                        [f64(W) for W in heads.W], tau, 1e-5, bf16)
        assert ref["exit_layer"].max() <= 2
        ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows)
        for repeat in range(2):                               # the second call meets the first one's leftovers
            ex = torch.full((rows,), -1, dtype=torch.int32, device=DEV)
            tok = torch.full((rows,), -1, dtype=torch.int32, device=DEV)
            Hout = torch.full((5, rows), 7.0, device=DEV)
            nev = torch.zeros(1, dtype=torch.int64, device=DEV)
            B.eh_cascade(ctx, hid.h, rows, ex, tok, Hout, nev)
            torch.cuda.synchronize()
            B.eh_check(ctx)
            np.testing.assert_array_equal(ex.cpu().numpy(), ref["exit_layer"], err_msg=name)
            bad = np.flatnonzero(tok.cpu().numpy() != ref["token"])
            assert all(ref["gap"][ref["exit_layer"][r], r] < P.NEAR_TIE for r in bad), name
            Hg = Hout.double().cpu().numpy()
            seen = ~np.isnan(ref["H"])
            np.testing.assert_array_equal(~np.isnan(Hg), seen, err_msg=name)
            assert np.abs(Hg[seen] - ref["H"][seen]).max() <= P.TOL_H
            assert int(nev.item()) == int(seen.sum()) == int((ref["exit_layer"] + 1).sum())
        B.eh_destroy(ctx)


# ------------------------------------------------------------------ NaN / Inf hidden states
@pytest.mark.parametrize("dtype,rows", [("bf16", 40), ("bf16", 150), ("bf16", 9), ("f32", 40), ("f32", 9)])
def test_nan_and_inf_rows_have_defined_outputs(B, dtype, rows):
    """A hidden state with a NaN or an Inf in it: NaN entropy and log-sum-exp, argmax -1, never
    through the exit test; every other row is untouched.  The oracle says the same."""
    bf16 = dtype == "bf16"
    w = G.Workload("nan", d=128, V=3000, n_heads=3, rows=rows, dtype=dtype, seed=rows + 77, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    bad_nan, bad_inf, bad_last = 2, rows - 1, 5
    hid.h[0, bad_nan, 17] = float("nan")
    hid.h[0, bad_inf, 0] = float("inf")
    hid.h[1, bad_inf, 3] = float("-inf")
    hid.h[:, bad_last, 100] = float("nan")                    # NaN at every head: token -1 at the last
    tau = [1e9, 1e9, float("inf")]                              # every finite entropy exits at head 0
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows)
    for l in range(3):
        H, lse, am = _outs(rows)
        B.eh_eval(ctx, l, hid.h[l], rows, H, lse, am)
        torch.cuda.synchronize()
        orc = P.oracle_head(hid.h[l], heads.gamma[l], heads.beta[l], heads.W[l], bf16)
        nan_o = np.isnan(orc[0])
        assert nan_o.sum() == (3 if l == 0 else 2 if l == 1 else 1)
        np.testing.assert_array_equal(torch.isnan(H).cpu().numpy(), nan_o)
        np.testing.assert_array_equal(torch.isnan(lse).cpu().numpy(), nan_o)
        assert (am.cpu().numpy()[nan_o] == -1).all() and (orc[2][nan_o] == -1).all()
        keep = torch.from_numpy(np.flatnonzero(~nan_o)).to(DEV)
        P.compare_head(f"nan/{dtype}/{rows}/head{l}", H[keep], lse[keep], am[keep], tuple(x[~nan_o] for x in orc), [])
    f64 = P.f64
    ref = O.cascade([f64(hid.h[l]) for l in range(3)], [f64(g) for g in heads.gamma], [f64(b) for b in heads.beta],
                    [f64(W) for W in heads.W], tau, 1e-5, bf16)
    assert ref["exit_layer"][bad_nan] == 1 and ref["exit_layer"][bad_inf] == 2 and ref["token"][bad_last] == -1
    ex = torch.full((rows,), -1, dtype=torch.int32, device=DEV)
    tok = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    B.eh_cascade(ctx, hid.h, rows, ex, tok, None, None)
    torch.cuda.synchronize()
    B.eh_check(ctx)
    np.testing.assert_array_equal(ex.cpu().numpy(), ref["exit_layer"])
    badtok = np.flatnonzero(tok.cpu().numpy() != ref["token"])
    assert all(ref["gap"][ref["exit_layer"][r], r] < P.NEAR_TIE for r in badtok)
    assert int(tok[bad_last].item()) == -1
    B.eh_destroy(ctx)


@pytest.mark.parametrize("Bsz,k", [(2, 3), (6, 4)])
def test_verify_with_a_nan_position(B, Bsz, k):
    rows = Bsz * (k + 1)
    w = G.Workload("nanver", d=128, V=3000, n_heads=1, rows=rows, dtype="bf16", seed=rows)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV, amp=torch.full((rows,), 1.5))
    f_final = hid.h[0].reshape(Bsz, k + 1, w.d).contiguous()
    f_final[1, 2, 9] = float("nan")
    f64 = P.f64
    _, _, tgt0, _ = O.dssd_verify(f64(f_final), np.zeros((Bsz, k), dtype=np.int64), f64(heads.gamma[0]),
                                  f64(heads.beta[0]), f64(heads.W[0]), None, 1e-5, True)
    draft = tgt0[:, :k].copy()                                  # all drafts right: row 1 stops at the NaN position
    draft[1, 2] = 0
    acc_o, nxt_o, tgt_o, gap_o = O.dssd_verify(f64(f_final), draft, f64(heads.gamma[0]), f64(heads.beta[0]),
                                               f64(heads.W[0]), None, 1e-5, True)
    assert tgt_o[1, 2] == -1 and acc_o[1] == 2 and nxt_o[1] == -1 and acc_o[0] == k
    assert np.nanmin(gap_o) > 1e-3
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [float("inf")], max_rows=rows)
    acc = torch.full((Bsz,), -5, dtype=torch.int32, device=DEV)
    nxt = torch.full((Bsz,), -5, dtype=torch.int32, device=DEV)
    tgt = torch.full((Bsz, k + 1), -5, dtype=torch.int32, device=DEV)
    B.dssd_verify(ctx, f_final, torch.from_numpy(draft).to(torch.int32).to(DEV).contiguous(), None, acc, nxt, tgt)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(tgt.cpu().numpy(), tgt_o)
    np.testing.assert_array_equal(acc.cpu().numpy(), acc_o)
    np.testing.assert_array_equal(nxt.cpu().numpy(), nxt_o)
    B.eh_destroy(ctx)


# ------------------------------------------------------------------ the persistent kernel gives up and recovers
def test_persistent_kernel_gives_up_cleanly_and_recovers(B):
    """With the bound of its waits set to zero polls a workgroup gives up at the first record of
    another workgroup that is not there yet: every kernel still ends, eh_check reports the failure
    once, rows that were not finished read -1 / NaN, and the next call on the context is normal."""
    w = G.scaled(G.CONFIGS["c1_decode"], n_heads=6, rows=8)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    tau = G.tau_linear(w)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=8)

    def cascade():
        ex = torch.full((8,), -7, dtype=torch.int32, device=DEV)
        tok = torch.full((8,), -7, dtype=torch.int32, device=DEV)
        Hout = torch.full((6, 8), 5.0, device=DEV)
        B.eh_cascade(ctx, hid.h, 8, ex, tok, Hout, None)
        torch.cuda.synchronize()
        return ex.cpu().numpy(), tok.cpu().numpy(), Hout.cpu().numpy()

    good = cascade()
    B.eh_check(ctx)
    assert (good[0] >= 0).all() and (good[1] >= 0).all()
    B.eh_set_spin_limit(ctx, 0)
    failures = 0
    for _ in range(3):
        ex, tok, Hout = cascade()
        try:
            B.eh_check(ctx)
        except B.EhError as e:
            failures += 1
            assert e.status == 5
        for r in range(8):                                    # finished rows are right, the others preset
            assert (ex[r], tok[r]) in ((-1, -1), (good[0][r], good[1][r]))
        same = (Hout == good[2]) | (np.isnan(Hout))
        assert same.all()
        B.eh_check(ctx)                                       # reported once, then cleared
    assert failures >= 1, "zero polls never made a workgroup give up"
    H, lse, am = _outs(8)
    B.eh_eval(ctx, 2, hid.h[2], 8, H, lse, am)                # evaluation mode presets NaN / -1
    torch.cuda.synchronize()
    try:
        B.eh_check(ctx)
        assert torch.isfinite(H).all() and (am >= 0).all()
    except B.EhError:
        assert ((am == -1) | (am >= 0)).all() and (torch.isnan(H) | torch.isfinite(H)).all()
    B.eh_set_spin_limit(ctx, 1 << 22)
    again = cascade()
    B.eh_check(ctx)
    assert all(np.array_equal(a, b, equal_nan=True) for a, b in zip(good, again))
    with pytest.raises(B.EhError):
        B.eh_set_spin_limit(ctx, -1)
    B.eh_destroy(ctx)


@pytest.mark.parametrize("mode", ["cascade", "verify"])
def test_rows_kernel_gives_up_cleanly_and_recovers(B, mode):
    """The same for the persistent kernel behind 17 .. 64 rows (cascade and verification)."""
    w = G.Workload("giveup", d=256, V=20000, n_heads=5, rows=48, dtype="bf16", seed=8, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, G.tau_linear(w), max_rows=48)
    f_final = hid.h[4].reshape(6, 8, w.d).contiguous()
    gen = torch.Generator(device="cpu")
    gen.manual_seed(1)
    draft = torch.randint(0, w.V, (6, 7), generator=gen).to(torch.int32).to(DEV)

    def run():
        if mode == "cascade":
            a = torch.full((48,), -7, dtype=torch.int32, device=DEV)
            b = torch.full((48,), -7, dtype=torch.int32, device=DEV)
            B.eh_cascade(ctx, hid.h, 48, a, b, None, None)
        else:
            a = torch.full((6,), -7, dtype=torch.int32, device=DEV)
            b = torch.full((6,), -7, dtype=torch.int32, device=DEV)
            B.dssd_verify(ctx, f_final, draft, None, a, b, None)
        torch.cuda.synchronize()
        return a.cpu().numpy(), b.cpu().numpy()

    good = run()
    B.eh_check(ctx)
    assert (good[0] >= 0).all() and (good[1] >= 0).all()
    B.eh_set_spin_limit(ctx, 0)
    failures = 0
    for _ in range(3):
        a, b = run()
        try:
            B.eh_check(ctx)
        except B.EhError as e:
            failures += 1
            assert e.status == 5
        for i in range(len(a)):                               # finished rows are right, the others preset
            assert (a[i], b[i]) in ((-1, -1), (good[0][i], good[1][i]))
    assert failures >= 1, "zero polls never made a workgroup give up"
    B.eh_set_spin_limit(ctx, 1 << 22)
    again = run()
    B.eh_check(ctx)
    assert np.array_equal(good[0], again[0]) and np.array_equal(good[1], again[1])
    B.eh_destroy(ctx)


# ------------------------------------------------------------------ calibration level met exactly
def test_calibrate_level_at_the_boundary(B):
    w = G.Workload("calib", d=64, V=64, n_heads=1, rows=4, dtype="bf16", seed=1)
    heads = G.make_heads(w, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [float("inf")], max_rows=4)
    for eps, n, c in ((0.7, 10, 7), (0.01, 100, 1), (0.55, 20, 11), (0.02, 50, 1), (0.07, 100, 7), (0.4, 5, 2),
                      (0.3, 10, 3), (0.1, 10, 1), (0.9, 10, 9), (0.6, 5, 3), (1.0, 9, 9)):
        levels = [eps, min(1.0, float(np.nextafter(eps, 2.0))), float(np.nextafter(eps, -1.0))]
        for correct in (c, c - 1):
            H = torch.full((n,), 1.25, device=DEV)
            ref = torch.zeros(n, dtype=torch.int32, device=DEV)
            pred = torch.tensor([0] * correct + [1] * (n - correct), dtype=torch.int32, device=DEV)
            tau = torch.zeros(3, device=DEV)
            cnt = torch.zeros(3, dtype=torch.int64, device=DEV)
            B.eh_calibrate(ctx, H, pred, ref, levels, tau, cnt)
            torch.cuda.synchronize()
            t = O.correctness(pred.cpu().numpy(), ref.cpu().numpy())
            for i, e in enumerate(levels):
                want = O.calibrate_threshold(H.double().cpu().numpy(), t, e)
                assert (float(tau[i]), int(cnt[i])) == want, (eps, n, correct, i)
    B.eh_destroy(ctx)


# ------------------------------------------------------------------ few rows, hidden size above 2048
@pytest.mark.parametrize("rows", [1, 9, 16])
def test_few_rows_of_a_wide_model_run_the_persistent_cascade(B, rows):
    """The single-launch kernel for at most 16 rows stops at hidden size 2048; beyond it (the 2.8B
    shape of the batched configurations has 2560) a cascade or a verification of few rows is served
    by the persistent kernel for more rows, in one launch as well.  Parity as for any cascade; that it is
    that kernel which ran shows in its bounded wait giving up when told to poll zero times."""
    w = G.Workload("wide", d=2176, V=3000, n_heads=5, rows=rows, dtype="bf16", seed=40 + rows, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    n = w.n_heads
    full = P.oracle_all_heads(heads, hid.h, True)
    tau = G.tau_for_schedule(full[0], n) if rows > 1 else G.tau_linear(w)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows)
    ex = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    tok = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    Hout = torch.zeros((n, rows), device=DEV)
    nev = torch.zeros(1, dtype=torch.int64, device=DEV)
    B.eh_cascade(ctx, hid.h, rows, ex, tok, Hout, nev)
    torch.cuda.synchronize()
    B.eh_check(ctx)
    P.compare_cascade(f"wide{rows}", ex, tok, Hout, full[0], full[2], full[3], tau, [])
    assert int(nev.item()) == int((ex.long() + 1).sum().item())
    # verification of the same rows as one draft row of rows - 1 tokens (final head)
    k = rows - 1
    fin = n - 1
    f_final = hid.h[fin].reshape(1, rows, w.d).contiguous()
    target_o = full[2][fin]                                          # the oracle's argmax per position
    draft = torch.tensor(target_o[:k].reshape(1, k), dtype=torch.int32, device=DEV)
    if k >= 3:
        draft[0, k // 2] = (int(target_o[k // 2]) + 1) % w.V          # first mismatch in the middle
    acc = torch.full((1,), -7, dtype=torch.int32, device=DEV)
    nxt = torch.full((1,), -7, dtype=torch.int32, device=DEV)
    tgt = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    B.dssd_verify(ctx, f_final, draft, None, acc, nxt, tgt)
    torch.cuda.synchronize()
    B.eh_check(ctx)
    near = full[3][fin] < P.NEAR_TIE
    assert all(int(tgt[i]) == int(target_o[i]) or near[i] for i in range(rows))
    if not near.any():
        want = k // 2 if k >= 3 else k
        assert int(acc.item()) == want and int(nxt.item()) == int(target_o[want])
    # the persistent kernel, not the launch-per-head path: only it can give up
    B.eh_set_spin_limit(ctx, 0)
    gave_up = 0
    for _ in range(3):
        B.eh_cascade(ctx, hid.h, rows, ex, tok, None, None)
        try:
            B.eh_check(ctx)
        except B.EhError:
            gave_up += 1
    assert gave_up >= 1
    B.eh_set_spin_limit(ctx, 1 << 22)
    ex2 = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    tok2 = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    B.eh_cascade(ctx, hid.h, rows, ex2, tok2, None, None)
    torch.cuda.synchronize()
    B.eh_check(ctx)
    P.compare_cascade(f"wide{rows}b", ex2, tok2, None, full[0], full[2], full[3], tau, [])
    B.eh_destroy(ctx)


# ------------------------------------------------------------------ every block layout of a cascade
@pytest.mark.parametrize("rows", [17, 33, 97, 129, 161, 193, 225, 256])
def test_cascade_across_block_layouts(B, rows):
    """1 to 8 blocks of 32 rows: one and two on the persistent k-split kernel (17 and 33 rows), more on
    the eight waves of the batched kernel behind a cascade of two launches per head, a block or none per wave,
    shrinking from head to head as rows leave on the 10 / 40 / 70 % schedule; the oracle on every row, and the same call twice for a bitwise repeat (the
    list of live rows is built through atomics)."""
    w = G.Workload("blocks", d=160, V=2500, n_heads=7, rows=rows, dtype="bf16", seed=900 + rows, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    n = w.n_heads
    full = P.oracle_all_heads(heads, hid.h, True)
    tau = G.tau_for_schedule(full[0], n)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows)
    outs = []
    for _ in range(2):
        ex = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
        tok = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
        Hout = torch.zeros((n, rows), device=DEV)
        nev = torch.zeros(1, dtype=torch.int64, device=DEV)
        B.eh_cascade(ctx, hid.h, rows, ex, tok, Hout, nev)
        torch.cuda.synchronize()
        B.eh_check(ctx)
        outs.append((ex, tok, Hout, nev))
    ex, tok, Hout, nev = outs[0]
    P.compare_cascade(f"blocks{rows}", ex, tok, Hout, full[0], full[2], full[3], tau, [])
    assert int(nev.item()) == int((ex.long() + 1).sum().item())
    assert len(set(ex.tolist())) >= 4
    assert torch.equal(ex, outs[1][0]) and torch.equal(tok, outs[1][1])
    assert torch.equal(Hout.view(torch.int32), outs[1][2].view(torch.int32))
    B.eh_destroy(ctx)


# ------------------------------------------------------------------ the persistent kernel above 64 rows
@pytest.mark.parametrize("d,V,rows", [(4096, 16384, 65), (4096, 16384, 97), (4096, 16384, 103), (6656, 20000, 129),
                                      (6656, 20000, 171), (1024, 50304, 108), (64, 630000, 66), (640, 50304, 89), (960, 40001, 89),
                                      (288, 128256, 66)])
def test_persistent_cascade_above_64_rows(B, d, V, rows):
    """Where a head's stream is long, cascades of 65 to 26 + V (d + 620) / 10^6 rows run in one launch
    whose waves share weights through LDS: 3 to 7 blocks of 32 rows, one a wave of eight (the largest of each
    shape among them), shrinking as rows leave; LayerNorm in registers and (d above 4096) from memory;
    ties at the top, a NaN row, a bitwise repeat, and the bounded wait giving up, which shows that it is
    that kernel."""
    n, pair = 5, (100, 2900)
    w = G.Workload("rows65", d=d, V=V, n_heads=n, rows=rows, dtype="bf16", seed=60 + rows, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    full = P.oracle_all_heads(heads, hid.h, True)
    tau = G.tau_for_schedule(full[0], n)

    def cascade(ctx, want_H=True):
        ex = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
        tok = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
        H = torch.zeros((n, rows), device=DEV) if want_H else None
        nev = torch.zeros(1, dtype=torch.int64, device=DEV)
        B.eh_cascade(ctx, hid.h, rows, ex, tok, H, nev)
        torch.cuda.synchronize()
        return ex, tok, H, nev

    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows)
    a = cascade(ctx)
    B.eh_check(ctx)
    b = cascade(ctx)
    B.eh_check(ctx)
    P.compare_cascade(f"rows{rows}", *a[:3], full[0], full[2], full[3], tau, [])
    assert int(a[3]) == int((a[0].long() + 1).sum()) and len(set(a[0].tolist())) >= 4
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and torch.equal(a[2].view(torch.int32), b[2].view(torch.int32))
    # zero polls: only the persistent kernel can give up; finished rows are right, the others -1
    B.eh_set_spin_limit(ctx, 0)
    failures = 0
    for _ in range(3):
        ex, tok, _, _ = cascade(ctx, want_H=False)
        try:
            B.eh_check(ctx)
        except B.EhError as e:
            failures += 1
            assert e.status == 5
        done = ex >= 0
        assert torch.equal(ex[done], a[0][done]) and torch.equal(tok[done], a[1][done])
        assert (ex[~done] == -1).all() and (tok[~done] == -1).all()
    assert failures >= 1, "zero polls never made a workgroup give up"
    B.eh_set_spin_limit(ctx, 1 << 22)
    again = cascade(ctx)
    B.eh_check(ctx)
    assert torch.equal(a[0], again[0]) and torch.equal(a[1], again[1])
    B.eh_destroy(ctx)
    # ties at the top of head 0, where every row with a finite entropy leaves; a NaN row goes to the end
    wins = _plant_ties(w, heads, hid, [pair], True)[0]
    bad = rows - 2
    hid.h[:, bad, 7] = float("nan")
    orc = P.oracle_head(hid.h[0], heads.gamma[0], heads.beta[0], heads.W[0], True)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [1e9] * (n - 1) + [float("inf")], max_rows=rows)
    ex, tok, H, _ = cascade(ctx)
    B.eh_check(ctx)
    B.eh_destroy(ctx)
    keep = [r for r in range(rows) if r != bad]
    assert (ex[keep] == 0).all() and int(ex[bad]) == n - 1 and int(tok[bad]) == -1 and bool(torch.isnan(H[:, bad]).all())
    P.compare_head("rows tie", H[0, keep], torch.from_numpy(orc[1][keep]), tok[keep], tuple(x[keep] for x in orc), [])
    tied = [r for r in wins if r != bad and orc[3][r] == 0.0 and orc[2][r] == pair[0]]
    assert len(tied) >= 1 and all(int(tok[r]) == pair[0] for r in tied)


@pytest.mark.parametrize("d,V,rows", [(4096, 16384, 96), (6656, 20000, 104), (6656, 20000, 128), (6656, 20000, 161),
                                      (4096, 50304, 129), (4096, 50304, 193), (2048, 70000, 192), (2048, 70000, 193)])
def test_persistent_cascade_service_workgroups(B, d, V, rows):
    """One row per service wave or two: 12 to 24 workgroups of eight such waves, at the last row that a
    count takes and the first of the next, and the heads of 300 MB and more that keep two."""
    test_persistent_cascade_above_64_rows(B, d, V, rows)


# ------------------------------------------------------------------ live rows across groups of 256
@pytest.mark.parametrize("rows", [300, 400, 513])
def test_cascade_whose_live_rows_cross_256(B, rows):
    """The batched kernel shares its grid out between the groups of 256 rows that are live (here 2 or
    3, then fewer as rows leave), and kernel and merge work the number of partial statistics out on
    their own: V is large enough for the number to change with every group."""
    n = 6
    w = G.Workload("cross", d=64, V=9001, n_heads=n, rows=rows, dtype="bf16", seed=rows, kappa=0.6)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    full = P.oracle_all_heads(heads, hid.h, True)
    tau = G.tau_for_schedule(full[0], n)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, tau, max_rows=rows)
    ex = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    tok = torch.full((rows,), -7, dtype=torch.int32, device=DEV)
    for _ in range(2):                                        # the second call meets the first one's partials
        H = torch.zeros((n, rows), device=DEV)
        nev = torch.zeros(1, dtype=torch.int64, device=DEV)
        B.eh_cascade(ctx, hid.h, rows, ex, tok, H, nev)
        torch.cuda.synchronize()
        P.compare_cascade(f"cross{rows}", ex, tok, H, full[0], full[2], full[3], tau, [])
        assert int(nev) == int((ex.long() + 1).sum())
    live = [int((ex >= l).sum()) for l in range(n)]
    assert len({(x + 255) // 256 for x in live}) >= 2, live
    B.eh_destroy(ctx)


def test_eval_at_live_counts_around_256(B):
    R = 400
    w = G.Workload("live256", d=64, V=9001, n_heads=1, rows=R, dtype="bf16", seed=12)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    orc = P.oracle_head(hid.h[0], heads.gamma[0], heads.beta[0], heads.W[0], True)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0], max_rows=R)
    idx = torch.randperm(R, generator=torch.Generator().manual_seed(4)).to(torch.int32)
    for n in (0, 1, 255, 256, 257, 400):
        H, lse, am = _outs(R)
        B.eh_eval(ctx, 0, hid.h[0], R, H, lse, am, row_idx=idx.to(DEV), n_rows_dev=torch.tensor([n], dtype=torch.int32, device=DEV))
        torch.cuda.synchronize()
        if n:
            P.compare_head(f"live{n}", H[:n], lse[:n], am[:n], tuple(x[idx[:n].numpy()] for x in orc), [])
        assert bool(torch.isnan(H[n:]).all()) and bool(torch.isnan(lse[n:]).all()) and bool((am[n:] == -7).all())
    B.eh_destroy(ctx)


# ------------------------------------------------------------------ the weight ring across passes and heads
@pytest.mark.parametrize("d,rows,V", [(8, 90, 3001), (32, 520, 50304), (64, 40, 57000), (64, 300, 9001), (96, 70, 50304), (128, 300, 50304), (160, 129, 3001), (192, 300, 50304),
                                      (224, 256, 70001), (256, 65, 50257), (544, 520, 20000)])
def test_weights_run_on_from_pass_to_pass(B, d, rows, V):
    """Two heads on 40 to 520 rows.  The ring of weights runs on from pass to pass and head to head where
    a pass has at least 6 k-steps of 32 (d > 160) and is filled anew below; a pass has at least three k-steps
    (narrower heads run the missing ones without activations), and their number modulo 3 decides which
    steps come first.  Slices of one to
    three passes, of unequal lengths; one to three groups of rows, the last waves without a block."""
    w = G.Workload("ring", d=d, V=V, n_heads=2, rows=rows, dtype="bf16", seed=d + rows)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0, 0.0], max_rows=rows)
    out = [torch.zeros((2, rows), device=DEV) for _ in range(4)]
    am = torch.full((2, rows), -7, dtype=torch.int32, device=DEV)
    B.eh_eval_heads_metrics(ctx, 0, 2, hid.h, rows, out[0], out[1], am, out[2], out[3])
    for l in range(2):
        P.compare_head(f"ring{d}/{l}", out[0][l], out[1][l], am[l],
                       P.oracle_head(hid.h[l], heads.gamma[l], heads.beta[l], heads.W[l], True), [])
        one = _outs(rows)                             # the bits do not depend on what is evaluated around a head
        B.eh_eval(ctx, l, hid.h[l], rows, *one)
        assert torch.equal(one[0], out[0][l]) and torch.equal(one[1], out[1][l]) and torch.equal(one[2], am[l])
    n = rows - rows // 3                              # fewer live rows than the host knows of
    live = _outs(rows)
    B.eh_eval(ctx, 1, hid.h[1], rows, *live, n_rows_dev=torch.tensor([n], dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    P.compare_head(f"ring{d}/live", live[0][:n], live[1][:n], live[2][:n],
                   P.oracle_head(hid.h[1][:n], heads.gamma[1], heads.beta[1], heads.W[1], True), [])
    assert bool(torch.isnan(live[0][n:]).all())
    B.eh_destroy(ctx)


@pytest.mark.parametrize("rows", [128, 512])
def test_narrow_heads_take_no_longer_than_wider_ones(B, rows):
    """Heads of fewer k-steps than a pass has go the same way as those next to them: 8 heads of d = 32 and 64
    took three times as long as of d = 96 where they went another."""
    times = {}
    for d in (32, 64, 96):
        w = G.Workload("narrow", d=d, V=50304, n_heads=8, rows=rows, dtype="bf16", seed=d)
        heads = G.make_heads(w, DEV)
        ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0] * 8, max_rows=rows)
        h = torch.randn((8, rows, d), device=DEV).to(torch.bfloat16)
        H, lse = torch.zeros((8, rows), device=DEV), torch.zeros((8, rows), device=DEV)
        am = torch.zeros((8, rows), dtype=torch.int32, device=DEV)
        turns = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                B.eh_eval_heads(ctx, 0, 8, h, rows, H, lse, am)
            b.record()
            torch.cuda.synchronize()
            turns.append(a.elapsed_time(b))
        times[d] = sorted(turns)[2]
        B.eh_destroy(ctx)
    assert times[32] < 1.3 * times[96] and times[64] < 1.3 * times[96], times


@pytest.mark.parametrize("d,rows,V", [(32, 70, 9001), (64, 300, 50304), (96, 33, 50304), (224, 520, 20000)])
def test_losses_of_narrow_heads(B, d, rows, V):
    """The dual pass has at least three k-steps: a head of d <= 64 runs the missing ones without activations."""
    w = G.Workload("duo", d=d, V=V, n_heads=2, rows=rows, dtype="bf16", seed=d + rows)
    heads = G.make_heads(w, DEV)
    hid = G.make_hidden(w, heads, DEV)
    labels = torch.randint(0, V, (rows,), generator=torch.Generator().manual_seed(d), dtype=torch.int32)
    ctx = B.eh_create(heads.W, heads.gamma, heads.beta, [0.0, 0.0], max_rows=rows)
    kl, ce, loss = torch.zeros(rows, device=DEV), torch.zeros(rows, device=DEV), torch.zeros(3, device=DEV)
    B.eh_head_losses(ctx, 0, hid.h[0], hid.h[1], labels.to(DEV), rows, 0.3, kl, ce, loss)
    torch.cuda.synchronize()
    f = P.f64
    ref = O.head_losses(f(hid.h[0]), f(hid.h[1]), f(heads.gamma[0]), f(heads.beta[0]), f(heads.W[0]), f(heads.gamma[1]),
                        f(heads.beta[1]), f(heads.W[1]), labels.numpy(), 0.3, bf16=True)
    for got, key in ((kl, "kl"), (ce, "ce")):
        want = np.asarray(ref[key])
        # a logit is an fp32 sum of up to 224 exact products, 14 matrix steps of partial sums up to about 15:
        # sqrt(14) * 15 * 2^-24 = 3e-6, and the sums over V add roundings of that size; measured at most 3.1e-6
        assert np.all(np.abs(got.double().cpu().numpy() - want) <= 1e-5 + 1e-6 * np.abs(want)), key
    B.eh_destroy(ctx)


# ------------------------------------------------------------------ LayerNorm of many rows at once
@pytest.mark.parametrize("d,rows,heads", [(72, 130, 8), (520, 257, 4), (4096, 260, 4), (4104, 260, 4), (1000, 1000, 2), (96, 127, 8), (96, 96, 8)])
def test_layernorm_of_many_rows(B, d, rows, heads):
    """From 1024 rows of all heads together, each head's rows padded to 32, a wave normalises a row and eight rows go
    out together (hidden sizes up to 4096; 8 heads of 127 rows are exactly 1024, of 96 rows stay below).  Rows that do not fill the last eight, hidden sizes
    that do not fill a lane's share, rows further apart than d, and rows of zeros and of tiny values, whose
    outputs are no normal bf16 numbers before beta."""
    w = G.Workload("many", d=d, V=300, n_heads=heads, rows=rows, dtype="bf16", seed=d + rows)
    hs = G.make_heads(w, DEV)
    hid = G.make_hidden(w, hs, DEV)
    for l in range(heads):
        hs.beta[l][::3] = 0.0
    h = torch.full((heads, rows, d + 8), 3.0, dtype=torch.bfloat16, device=DEV)
    h[:, :, :d] = hid.h
    h[:, 1, :d] = 0.0                                 # no variance: y is beta, zero at every third place
    h[:, 2, :d] *= 1e-30
    ctx = B.eh_create(hs.W, hs.gamma, hs.beta, [0.0] * heads, max_rows=rows)
    H, lse = torch.zeros((heads, rows), device=DEV), torch.zeros((heads, rows), device=DEV)
    am = torch.full((heads, rows), -7, dtype=torch.int32, device=DEV)
    B.eh_eval_heads(ctx, 0, heads, h[:, :, :d], rows, H, lse, am)
    torch.cuda.synchronize()
    for l in range(heads):
        P.compare_head(f"many{d}/{l}", H[l], lse[l], am[l],
                       P.oracle_head(h[l, :, :d].contiguous(), hs.gamma[l], hs.beta[l], hs.W[l], True), [])
    B.eh_destroy(ctx)
