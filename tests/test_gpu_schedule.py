"""The forward work list at the edges of the scheduler's ranges, read back from the workspace: every (sequence, block, head)
once, whole or as pieces that tile its tile list, longest first.  Costs are recomputed from the mask's definition (dense causal:
a block of 128 query rows that ends at row r sees the 32-key tiles 0 .. r / 32)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = {                                       # lengths, heads
    "one-row": ([1], 1),
    "empty-between": ([0, 130, 0, 0, 1, 257, 0], 3),
    "wave-edge": ([128] * 63 + [129], 2),        # 65 blocks: one more than a wave counts at a time
    "cached-batch": ([40] * 1024, 1),            # batch of the size whose prefix sums fit in LDS
    "uncached-batch": ([40] * 1025, 1),
    "sort-limit": ([1024] * 1024, 1),            # 8,192 blocks: the longest list that is sorted
    "beyond-sort": ([1024] * 1024 + [1], 2),
    "cut": ([8192, 100, 3000], 2),               # few long blocks: cut along the key axis
    "wide-keys": ([140000, 5000], 1),            # more than 4,095 tiles: sorted by classes of 2 tiles
}


@pytest.mark.parametrize("name", list(CASES))
def test_forward_work_list(name):
    from paper_2602_16986_amd import binding as hb
    lengths, H = CASES[name]
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    T = int(off[-1])
    q = torch.zeros(T, H, 128, dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(q)
    offsets = torch.from_numpy(off).cuda()
    prob = hb.AttnProblem(q, q, q, out, offsets, max_seqlen=max(lengths), seq_offsets_host=off)
    ws = hb.new_workspace(hb.hstu_attn_workspace_bytes(prob, False), "cuda")
    ws.fill_(0xA5)
    hb.hstu_attn_fwd(prob, q, q, q, out, ws)
    torch.cuda.synchronize()
    st = hb.hstu_attn_schedule_stats(prob, ws, False)
    items = ws[256:256 + 32 * st["items"]].cpu().numpy().view(np.int32).reshape(-1, 8)
    count = {(b, rb): (min(128 * rb + 128, L) - 1) // 32 + 1 for b, L in enumerate(lengths) for rb in range((L + 127) // 128)}
    assert st["tiles"] == H * sum(count.values())
    cover, slots, costs = {}, [], []
    for b, rbh, t0, t1, slot, seq0, length, hist in items.tolist():
        assert (seq0, length, hist) == (int(off[b]), lengths[b], lengths[b])
        end = min(t1, count[(b, rbh >> 8)])
        cover.setdefault((b, rbh >> 8, rbh & 255), []).append((t0, end, slot))
        slots += [slot] if slot >= 0 else []
        costs.append(end - t0)
    assert set(cover) == {(b, rb, h) for (b, rb) in count for h in range(H)}
    assert len(slots) == len(set(slots))
    for key, v in cover.items():
        v.sort()
        assert v[0][0] == 0 and v[-1][1] == count[key[:2]] and all(x[1] == y[0] for x, y in zip(v, v[1:])), (key, v)
        assert (len(v) == 1) == (v[0][2] < 0), (key, v)
    if sum((L + 127) // 128 for L in lengths) <= 8192:
        shift = max(int(max(costs)).bit_length() - 12, 0)
        group = 4 * H
        firsts = [max(costs[i:i + group]) >> shift for i in range(0, len(costs), group)]
        lasts = [min(costs[i:i + group]) >> shift for i in range(0, len(costs), group)]
        assert all(a >= b for a, b in zip(lasts, firsts[1:])), "entries are not in longest-first order"
    assert (len(slots) > 0) == (name in ("cut", "wide-keys"))
    assert torch.count_nonzero(out) == 0
