"""Non-finite rows with 32 and 64 features per head, bf16: a row that a token may not see leaves that token's results as they are without it, bit for
bit.  Exactly so where the row enters through the scores (K in the forward, V in dQ, Q in dV, dO in dK); a row that is multiplied
by the probabilities themselves (V in the forward, K in dQ, Q in dK, dO in dV) may reach the other pairs of a block of 32 x 64 tokens that holds a
visible pair, since a matrix product multiplies it by their zeros, and no further."""
import numpy as np
import pytest
import torch

from paper_2602_16986_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = {                               # lengths, K1, K2, candidates, row that is not finite
    "dense": ([300, 129], -1, 0, None, (45, 100, 128, 250, 299, 330)),
    "window": ([420, 70], 64, 0, None, (0, 31, 130, 300, 415)),
    "prefix": ([700], 130, 70, None, (10, 69, 75, 127, 400)),
    "candidates": ([333, 97], -1, 0, [40, 97], (100, 292, 293, 300, 332, 340)),
    "window-candidates": ([500], 90, 33, [120], (20, 200, 340, 379, 380, 450)),
}


def visible_pairs(w):
    """[T, T] truth values of the mask: query row, key column."""
    vis = np.zeros((w.T, w.T), dtype=bool)
    for b in range(len(w.lengths)):
        o, L = int(w.offsets[b]), int(w.lengths[b])
        n = L - (0 if w.num_targets is None else int(w.num_targets[b]))
        i, j = np.arange(L)[:, None], np.arange(L)[None, :]
        p = np.minimum(i, n)
        seen = (j < n) & (j <= p)
        if w.K1 >= 0:
            seen &= (p - j < w.K1) | (j < w.K2)
        vis[o:o + L, o:o + L] = seen | ((i >= n) & (i == j))
    return vis


def near(w, vis, mine, other):
    """Pairs of the blocks (mine x other tokens from the start of a sequence) that hold a visible pair."""
    out = np.zeros_like(vis)
    for b in range(len(w.lengths)):
        o, L = int(w.offsets[b]), int(w.lengths[b])
        for i in range(o, o + L, mine):
            for j in range(o, o + L, other):
                ie, je = min(i + mine, o + L), min(j + other, o + L)
                out[i:ie, j:je] = vis[i:ie, j:je].any()
    return out


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("d", [32, 64])
def test_masked_rows_that_are_not_finite(d, name, value):
    from paper_2602_16986_amd.runner import DeviceWorkload
    lengths, K1, K2, targets, rows = CASES[name]
    w = wl.build(name, lengths, 2, d, "bf16", seed=3, K1=K1, K2=K2, backward=True,
                 num_targets=None if targets is None else np.array(targets, dtype=np.int32))
    vis = visible_pairs(w)
    by_query, by_key = near(w, vis, 32, 64), near(w, vis, 64, 32)
    dw = DeviceWorkload(w)

    def results():
        for t in (dw.out, dw.dq, dw.dk, dw.dv):
            t.fill_(float("nan"))
        dw.attn_fwd()
        dw.attn_bwd()
        torch.cuda.synchronize()
        return {"A": dw.out.clone(), "dQ": dw.dq.clone(), "dK": dw.dk.clone(), "dV": dw.dv.clone()}
    clean = results()
    # operand -> result -> pairs over which the row may show
    reach = {"k": {"A": vis, "dQ": by_query}, "v": {"A": by_query, "dQ": vis}, "q": {"dK": by_key, "dV": vis}, "dout": {"dK": vis, "dV": by_key}}
    for operand, on in reach.items():
        t = getattr(dw, operand)
        for r in rows:
            keep = t[r].clone()
            t[r] = value
            got = results()
            t[r] = keep
            for what, pairs in on.items():
                touched = pairs[:, r] if operand in ("k", "v") else pairs[r, :]
                if w.num_targets is not None and pairs is not vis:
                    # blocks that hold both kinds of rows are not told apart from visible ones: everything in the row's sequence
                    b = np.searchsorted(w.offsets, r, side="right") - 1
                    touched = np.zeros_like(touched)
                    touched[w.offsets[b]:w.offsets[b + 1]] = True
                free = torch.from_numpy(np.flatnonzero(~touched)).cuda()
                assert torch.equal(got[what][free], clean[what][free]), (operand, r, what)
