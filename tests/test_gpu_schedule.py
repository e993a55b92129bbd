"""The forward work list at the edges of the scheduler's ranges, read back from the workspace: every (sequence, block, head)
once, whole or as pieces that tile its tile list, longest first.  Costs are recomputed from the mask's definition (dense causal:
a block of 128 query rows that ends at row r sees the 32-key tiles 0 .. r / 32)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="session")
def plan(tmp_path_factory):
    """What the cut rule makes of a list, from the host check of the very header that the scheduler compiles."""
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_16986_amd", "csrc")
    so = str(tmp_path_factory.mktemp("plan") / "libplan.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(csrc, "geometry_check.cpp")])
    lib = ctypes.CDLL(so)

    def planned(lengths, targets, H, K1, K2, which, fp32, D):
        lengths = np.asarray(lengths, dtype=np.int32)
        targets = None if targets is None else np.asarray(targets, dtype=np.int32)
        costs, out = np.zeros(int(((lengths + 127) // 128).sum()), dtype=np.int32), (ctypes.c_int64 * 5)()
        tile = 64 if which == 1 and D == 128 and not fp32 else 32
        ptr = lambda a: None if a is None else a.ctypes.data_as(ctypes.c_void_p)
        lib.planned_list(len(lengths), ptr(lengths), ptr(targets), H, K1, K2, which, tile, int(fp32), D, ptr(costs), out)
        keys = [(b, rb) for b, L in enumerate(lengths) for rb in range((int(L) + 127) // 128 - 1, -1, -1)]
        return dict(zip(keys, costs.tolist())), dict(zip(("cut", "first", "chunk", "slots", "split"), out))
    return planned


def read_list(ws, T, B, H, fp32, second):
    """(header, items) of the first or the second list in a workspace; header: items, cut blocks, piece size."""
    blocks = (T // 128 + B) * H
    up = lambda n: (n + 255) // 256 * 256
    at = 256 + up((blocks + min((8 if fp32 else 2) * blocks, 768)) * 32) + up((B + 1) * 4) if second else 0
    head = ws[at:at + 32].cpu().numpy().view(np.int32)
    items = ws[at + 256:at + 256 + 32 * int(head[0])].cpu().numpy().view(np.int32).reshape(-1, 8)
    return {"items": int(head[0]), "split": int(head[1]), "chunk": int(head[6])}, items

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


RULE = {                                        # dtype, width, lengths, heads, K1, K2, candidates; whether the forward, dQ and dK/dV lists are cut
    "short-128": ("bf16", 128, [660, 100, 90, 80, 200], 2, -1, 0, None, (0, 0, 0)),
    "key-blocks-128": ("bf16", 128, [700, 100, 90, 80, 200], 2, -1, 0, None, (0, 0, 1)),
    "all-128": ("bf16", 128, [860, 100, 90, 80, 200], 2, -1, 0, None, (1, 1, 1)),
    "short-64": ("bf16", 64, [720, 100, 90, 80, 200], 2, -1, 0, None, (0, 0, 0)),
    "all-64": ("bf16", 64, [800, 100, 90, 80, 200], 2, -1, 0, None, (1, 1, 1)),
    "short-32": ("bf16", 32, [720, 100, 90, 80, 200], 2, -1, 0, None, (0, 0, 0)),
    "all-32": ("bf16", 32, [800, 100, 90, 80, 200], 2, -1, 0, None, (1, 1, 1)),
    "prefix-below": ("bf16", 128, [736] * 6, 2, 96, 200, None, (0, 0, 0)),
    "prefix-above": ("bf16", 128, [768] * 6, 2, 96, 200, None, (0, 0, 1)),
    "many-equal-blocks": ("bf16", 64, [1024] * 20, 4, -1, 0, None, (0, 0, 0)),
    "pieces-grow": ("bf16", 128, [3000], 2, -1, 0, None, (1, 1, 1)),
    "candidates": ("bf16", 64, [900, 100, 90, 200], 2, 100, 40, [50, 0, 9, 200], (0, 0, 1)),
    "fp32-short": ("fp32", 64, [64] * 3, 2, -1, 0, None, (0, 0, 0)),
    "fp32-cut": ("fp32", 64, [128] * 3, 2, -1, 0, None, (1, 1, 1)),
    "fp32-128": ("fp32", 128, [300, 70], 3, 40, 70, None, (1, 1, 1)),
    "fp32-32-short": ("fp32", 32, [224] * 4, 2, -1, 0, None, (0, 0, 1)),
    "fp32-32": ("fp32", 32, [256] * 4, 2, -1, 0, None, (1, 1, 1)),
}


@pytest.mark.parametrize("name", list(RULE))
def test_lists_against_the_cut_rule(name, plan):
    """All three lists on either side of the rule's thresholds: cut if and only if the rule says so, into the pieces and slots it says; every (sequence,
    block, head) once, whole or as pieces that tile its cost."""
    from paper_2602_16986_amd import binding as hb
    dtype, d, lengths, H, K1, K2, targets, expected = RULE[name]
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    T, B, fp32 = int(off[-1]), len(lengths), dtype == "fp32"
    q = torch.zeros(T, H, d, dtype=torch.float32 if fp32 else torch.bfloat16, device="cuda")
    dq, dk, dv, out = (torch.empty_like(q) for _ in range(4))
    tg = None if targets is None else torch.tensor(targets, dtype=torch.int32, device="cuda")
    prob = hb.AttnProblem(q, q, q, out, torch.from_numpy(off).cuda(), max_seqlen=max(lengths), seq_offsets_host=off, num_targets=tg, local_window=K1,
                          global_prefix=K2)
    ws_fwd, ws_bwd = (hb.new_workspace(hb.hstu_attn_workspace_bytes(prob, bwd), "cuda") for bwd in (False, True))
    for t in (ws_fwd, ws_bwd):
        t.fill_(0xA5)
    hb.hstu_attn_fwd(prob, q, q, q, out, ws_fwd)
    hb.hstu_attn_bwd(prob, q, q, q, q, dq, dk, dv, ws_bwd)
    torch.cuda.synchronize()
    for which in range(3):
        costs, rule = plan(lengths, targets, H, K1, K2, which, fp32, d)
        assert rule["cut"] == expected[which], (which, rule)
        head, items = read_list(ws_fwd if which == 0 else ws_bwd, T, B, H, fp32, which == 2)
        cover, slots = {}, []
        for b, rbh, t0, t1, slot, *_ in items.tolist():
            cover.setdefault((b, rbh >> 8, rbh & 255), []).append((t0, min(t1, costs[(b, rbh >> 8)]), slot))
            slots += [slot] if slot >= 0 else []
        assert set(cover) == {(b, rb, h) for (b, rb) in costs for h in range(H)}
        for key, v in cover.items():
            v.sort()
            assert v[0][0] == 0 and v[-1][1] == costs[key[:2]] and all(x[1] == y[0] for x, y in zip(v, v[1:])), (which, key, v)
            assert (len(v) == 1) == (v[0][2] < 0), (which, key, v)
        assert len(slots) == len(set(slots)) == (rule["slots"] if rule["cut"] else 0), (which, rule)
        assert head["split"] == (rule["split"] if rule["cut"] else 0), (which, rule, head)
        if rule["cut"]:
            assert head["chunk"] == rule["chunk"] and (name != "pieces-grow" or rule["chunk"] > rule["first"] or which == 1), (which, rule, head)
