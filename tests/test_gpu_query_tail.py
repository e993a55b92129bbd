"""Forward over a query tail: its blocks start at the 32 rows that hold the first wanted row, waves past the end of a sequence only load,
and pieces of the long key lists are added row by row.  Wanted rows against the oracle, all others untouched."""
import numpy as np
import pytest
import torch

from oracle import hstu_oracle as orc
from paper_2602_16986_amd import binding as hb
from paper_2602_16986_amd import workloads as wl
from test_gpu_parity import check, oracle_args, to_np, TOL

pytestmark = pytest.mark.gpu

LENGTHS = [1, 31, 32, 33, 64, 127, 128, 129, 160, 161, 1500, 2049]
TARGETS = [0, 31, 1, 2, 0, 100, 128, 1, 33, 0, 70, 129]


@pytest.mark.parametrize("dim,dtype", [(128, "bf16"), (64, "bf16"), (32, "fp32")])
@pytest.mark.parametrize("tail", [1, 31, 32, 33, 97, 4000])
@pytest.mark.parametrize("candidates", [False, True])
def test_tail_block_edges(dim, dtype, tail, candidates):
    targets = np.array(TARGETS, dtype=np.int32) if candidates else None
    K1, K2 = (200, 40) if candidates else (-1, 0)
    w = wl.build("tail-edges", LENGTHS, 2, dim, dtype, seed=11, K1=K1, K2=K2, num_targets=targets)
    from paper_2602_16986_amd.runner import DeviceWorkload
    dw = DeviceWorkload(w)
    prob = hb.AttnProblem(dw.q, dw.k, dw.v, dw.out, dw.offsets, max_seqlen=w.max_seqlen, num_targets=dw.num_targets, local_window=K1,
                          global_prefix=K2, alpha=w.alpha, inv_n=1.0 / w.N, rab_table=dw.table, rab_bounds=dw.bounds, query_tail=tail)
    ws = hb.new_workspace(hb.hstu_attn_workspace_bytes(prob, False), "cuda")
    ws.fill_(0xFF)                                          # NaNs: no partial sum may be read that was not written
    dw.out.fill_(7.0)
    hb.hstu_attn_fwd(prob, dw.q, dw.k, dw.v, dw.out, ws)
    torch.cuda.synchronize()
    got = to_np(dw.out)
    ref = orc.attn_fwd(w.q, w.k, w.v, w.offsets, **oracle_args(w))
    wanted = np.zeros(w.T, dtype=bool)
    for b, L in enumerate(LENGTHS):
        hist = L - (TARGETS[b] if candidates else 0)
        wanted[w.offsets[b] + max(hist - tail, 0):w.offsets[b] + L] = True
    check("A", got[wanted], ref[wanted], TOL[dtype])
    assert np.all(got[~wanted] == 7.0)


@pytest.mark.parametrize("dim,dtype", [(128, "bf16"), (32, "fp32")])
@pytest.mark.parametrize("lengths,tail", [([2600, 300], 700), ([3000, 2500], 500)])
def test_pieces_that_nearly_fit_their_slots(dim, dtype, lengths, tail):
    """Pieces of the first length take up to a quarter more slots than there are (114 of 96, 188 of 176); the next length is a quarter more."""
    from paper_2602_16986_amd.runner import DeviceWorkload
    w = wl.build("tail-pieces", lengths, 2, dim, dtype, seed=12)
    dw = DeviceWorkload(w)
    dw.problem.params.query_tail = tail
    dw.ws_fwd.fill_(0xFF)
    dw.out.fill_(7.0)
    dw.attn_fwd()
    torch.cuda.synchronize()
    items = hb.hstu_attn_schedule_stats(dw.problem, dw.ws_fwd)["items"]
    entries = dw.ws_fwd[256:256 + 32 * items].cpu().numpy().view(np.int32).reshape(-1, 8)
    assert (entries[:, 4] >= 0).any() and np.all(entries[entries[:, 4] >= 0][:, 3] - entries[entries[:, 4] >= 0][:, 2] <= 10)
    got = to_np(dw.out)
    ref = orc.attn_fwd(w.q, w.k, w.v, w.offsets, **oracle_args(w))
    wanted = np.concatenate([np.arange(L) >= L - tail for L in lengths])
    check("A", got[wanted], ref[wanted], TOL[dtype])
    assert np.all(got[~wanted] == 7.0)


@pytest.mark.parametrize("lengths,heads,least", [([20000], 1, 70), ([20000], 18, 33), ([9000, 9500], 1, 33), ([700, 5000, 1300], 1, 16), ([1500, 1100], 2, 2)])
def test_few_blocks_in_many_pieces(lengths, heads, least):
    """Up to 64 blocks, the longest in more pieces (and heads) than the scheduler has waves to share them, in fewer, or in few: pieces tile every
    block, and the wanted rows equal a float64 evaluation."""
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    gen, T, d, tail = torch.Generator(device="cuda").manual_seed(13), int(off[-1]), 128, 21
    q, k, v = (torch.randn(T, heads, d, generator=gen, device="cuda").mul(d ** -0.5).bfloat16() for _ in range(3))
    out = torch.full_like(q, 7.0)
    prob = hb.AttnProblem(q, k, v, out, torch.from_numpy(off).cuda(), max_seqlen=max(lengths), seq_offsets_host=off, inv_n=1.0 / max(lengths), query_tail=tail)
    ws = hb.new_workspace(hb.hstu_attn_workspace_bytes(prob, False), "cuda")
    ws.fill_(0xFF)
    hb.hstu_attn_fwd(prob, q, k, v, out, ws)
    torch.cuda.synchronize()
    items = ws[256:256 + 32 * hb.hstu_attn_schedule_stats(prob, ws, False)["items"]].cpu().numpy().view(np.int32).reshape(-1, 8)
    pieces = {}
    for b, rbh, t0, t1, slot, *_ in items.tolist():
        pieces.setdefault((b, rbh & 255), []).append((t0, t1, slot))
    assert len(pieces) == len(lengths) * heads and max(map(len, pieces.values())) >= least
    for (b, _), p in pieces.items():
        p.sort()
        assert p[0][0] == 0 and p[-1][1] >= -(-lengths[b] // 32) and all(x[1] == y[0] for x, y in zip(p, p[1:]))
        assert all(x[2] >= 0 for x in p) or len(p) == 1
    slots = [s for p in pieces.values() for _, _, s in p if s >= 0]
    assert len(slots) == len(set(slots))
    for b, L in enumerate(lengths):
        rows, seq = slice(off[b] + L - tail, off[b] + L), slice(off[b], off[b] + L)
        s = torch.matmul(q[rows].double().transpose(0, 1), k[seq].double().transpose(0, 1).transpose(1, 2).contiguous())
        seen = torch.arange(L, device="cuda")[None] <= torch.arange(L - tail, L, device="cuda")[:, None]
        ref = torch.matmul(torch.where(seen, s * torch.sigmoid(s), 0.0) / max(lengths), v[seq].double().transpose(0, 1).contiguous()).transpose(0, 1)
        check("A", to_np(out[rows]), ref.cpu().numpy(), TOL["bf16"])
        assert (out[off[b]:off[b] + L - tail] == 7.0).all()
