"""Kernel paths chosen by size, at the sizes where they can go wrong, against the oracle and, where
two paths must agree bit for bit, against each other."""
import numpy as np
import pytest
import torch

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
