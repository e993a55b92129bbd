"""The backward that hands dS from the dK/dV pass to the dQ product (bf16, 128 features): edges of its 32 x 128 tiles, of the key
blocks' query lists and of the 64-key steps, against the oracle; the same call in a workspace without room for dS, which takes two
independent passes; and a workspace sized from offsets that are not the device's."""
import numpy as np
import pytest
import torch

from oracle import hstu_oracle as orc
from paper_2602_16986_amd import binding as hb
from paper_2602_16986_amd import workloads as wl
from test_gpu_parity import check, oracle_args, to_np, TOL

pytestmark = pytest.mark.gpu

CASES = {                               # lengths, K1, K2, candidates
    "tile-edges": ([1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 257], -1, 0, None),
    "window-below-a-tile": ([300, 129, 1], 5, 0, None),
    "window-and-prefix": ([700, 513, 90], 130, 70, None),
    "prefix-only": ([400, 300], 0, 100, None),
    "prefix-only-candidates": ([400, 300, 131], 0, 100, [90, 0, 131]),
    "candidates": ([333, 97, 128, 260], -1, 0, [40, 97, 0, 132]),
    "window-candidates": ([600, 340], 64, 33, [250, 31]),
    "one-bucket-tiles": ([2600], -1, 0, None),
}


def workload(name):
    lengths, K1, K2, targets = CASES[name]
    return wl.build(name, lengths, 2, 128, "bf16", seed=3, K1=K1, K2=K2, backward=True,
                    num_targets=None if targets is None else np.array(targets, dtype=np.int32))


def backward(dw, ws):
    for t in (dw.dq, dw.dk, dw.dv):
        t.fill_(float("nan"))
    ws.fill_(0xFF)                      # bf16 NaNs: nothing may be read that was not written
    hb.hstu_attn_bwd(dw.problem, dw.q, dw.k, dw.v, dw.dout, dw.dq, dw.dk, dw.dv, ws)
    torch.cuda.synchronize()
    return [to_np(t) for t in (dw.dq, dw.dk, dw.dv)]


@pytest.mark.parametrize("name", list(CASES))
def test_backward_through_ds(name):
    from paper_2602_16986_amd.runner import DeviceWorkload
    w = workload(name)
    dw = DeviceWorkload(w, bias_grad=True)
    refs = orc.attn_bwd(w.q, w.k, w.v, w.dout, w.offsets, **oracle_args(w))
    ref_table = orc.attn_bwd_bias(w.q, w.k, w.v, w.dout, w.offsets, **oracle_args(w))
    full = hb.hstu_attn_workspace_bytes(dw.problem, True)
    by_length = dw.problem.params.seq_offsets_host
    for host_copy in (True, False):
        dw.problem.params.seq_offsets_host = by_length if host_copy else None
        size = hb.hstu_attn_workspace_bytes(dw.problem, True)
        assert size >= full
        dw.dtable.fill_(float("nan"))
        got = backward(dw, hb.new_workspace(size, "cuda"))
        for what, g, r in zip(("dQ", "dK", "dV"), got, refs):
            check(what, g, r, TOL["bf16"])
        check("dtable", to_np(dw.dtable), ref_table, TOL["bf16"])
    dw.problem.params.seq_offsets_host = by_length
    dw.dtable.fill_(float("nan"))
    got = backward(dw, hb.new_workspace(full - 256, "cuda"))          # 256 bytes short of the room for dS: two independent passes
    for what, g, r in zip(("dQ", "dK", "dV"), got, refs):
        check(what + " (no room)", g, r, TOL["bf16"])
    check("dtable (no room)", to_np(dw.dtable), ref_table, TOL["bf16"])


def test_least_workspace_is_accepted_and_no_less():
    from paper_2602_16986_amd.runner import DeviceLayer, DeviceWorkload
    w = workload("window-candidates")
    dw = DeviceWorkload(w)
    least = hb.hstu_attn_workspace_least_bytes(dw.problem, True)
    for what, g, r in zip(("dQ", "dK", "dV"), backward(dw, hb.new_workspace(least, "cuda")),
                          orc.attn_bwd(w.q, w.k, w.v, w.dout, w.offsets, **oracle_args(w))):
        check(what, g, r, TOL["bf16"])
    dl = DeviceLayer(wl.build_layer("least", [300, 129], 2, 128, 256, seed=4))
    dl.fwd()
    full = [t.float() for t in dl.bwd()]
    least_layer = hb.hstu_layer_workspace_least_bytes(dl.problem, True)
    assert least_layer < dl.ws_bwd.numel()
    dl.ws_bwd = hb.new_workspace(least_layer, "cuda")
    for a, b in zip(full, dl.bwd()):
        scale = float(a.abs().max())
        assert float((a - b.float()).abs().max()) <= TOL["bf16"] * scale
    for call, ws in ((lambda ws: backward(dw, ws), least), (lambda ws: (setattr(dl, "ws_bwd", ws), dl.bwd()), least_layer)):
        with pytest.raises(hb.HstuError) as e:
            call(hb.new_workspace(ws - 256, "cuda"))
        assert e.value.status == -4


@pytest.mark.parametrize("name", ["tile-edges", "window-and-prefix", "candidates", "one-bucket-tiles"])
@pytest.mark.parametrize("build_room,use_room,longer", [(False, True, 0), (True, False, 0), (False, True, 3000), (True, True, 3000)])
def test_lists_of_a_call_with_other_room(name, build_room, use_room, longer):
    """reuse_schedule between calls that decide differently about dS (a host copy of the offsets in one of them only, in a workspace that is
    too small without it) or that give another max_seqlen: the lists and the table of dS tiles lie where the second call looks for them."""
    from paper_2602_16986_amd.runner import DeviceWorkload
    w = workload(name)
    dw = DeviceWorkload(w, bias_grad=True)
    p = dw.problem.params
    host = p.seq_offsets_host
    sizes = []
    for extra in (0, longer):
        p.max_seqlen = w.max_seqlen + extra
        sizes.append(hb.hstu_attn_workspace_bytes(dw.problem, True))
    ws = hb.new_workspace(max(sizes), "cuda")
    refs = orc.attn_bwd(w.q, w.k, w.v, w.dout, w.offsets, **oracle_args(w))
    ref_table = orc.attn_bwd_bias(w.q, w.k, w.v, w.dout, w.offsets, **oracle_args(w))
    ws.fill_(0xFF)
    for call, (room, extra) in enumerate(((build_room, 0), (use_room, longer))):
        p.max_seqlen = w.max_seqlen + extra
        p.seq_offsets_host = host if room else None
        p.reuse_schedule = call
        size = sizes[call] if room else sizes[call] - 256
        outs = [torch.full_like(t, float("nan")) for t in (dw.q, dw.k, dw.v)]
        dw.dtable.fill_(float("nan"))
        hb.hstu_attn_bwd(dw.problem, dw.q, dw.k, dw.v, dw.dout, *outs, ws[:size])
        torch.cuda.synchronize()
        for what, g, r in zip(("dQ", "dK", "dV", "dtable"), [*outs, dw.dtable], [*refs, ref_table]):
            check(f"{what} (call {call})", to_np(g), r, TOL["bf16"])


def test_room_for_other_lengths_computes_nothing():
    """The host's copy of the offsets says sixteen short sequences, the device's say one long one that needs more room for dS: an empty
    list and untouched outputs, not a write behind the workspace."""
    T, H = 4096, 1
    host = np.arange(0, T + 1, 256, dtype=np.int32)
    device = np.zeros_like(host)
    device[1:] = T
    q = torch.randn(T, H, 128, device="cuda").to(torch.bfloat16)
    dq, dk, dv = (torch.full_like(q, 5.0) for _ in range(3))
    prob = hb.AttnProblem(q, q, q, q, torch.from_numpy(device).cuda(), max_seqlen=T, seq_offsets_host=host)
    ws = hb.new_workspace(hb.hstu_attn_workspace_bytes(prob, True), "cuda")
    hb.hstu_attn_bwd(prob, q, q, q, q, dq, dk, dv, ws)
    torch.cuda.synchronize()
    assert all(torch.all(t == 5.0) for t in (dq, dk, dv))


@pytest.mark.parametrize("dim,dtype,room", [(128, "bf16", True), (128, "bf16", False), (64, "bf16", False), (32, "fp32", False)])
def test_bias_gradient_with_one_copy_of_the_sums(dim, dtype, room):
    """max_seqlen so large that the sums per distance are kept once for the chip instead of once per die."""
    from paper_2602_16986_amd.runner import DeviceWorkload
    w = wl.build("one-copy", [700, 301, 64], 2, dim, dtype, seed=9, K1=400, K2=30, backward=True, num_targets=np.array([40, 0, 64], np.int32))
    dw = DeviceWorkload(w, bias_grad=True)
    dw.problem.params.max_seqlen = 300000
    size = hb.hstu_attn_workspace_bytes(dw.problem, True) if room else hb.hstu_attn_workspace_least_bytes(dw.problem, True)
    dw.dtable.fill_(float("nan"))
    got = backward(dw, hb.new_workspace(size, "cuda"))
    for what, g, r in zip(("dQ", "dK", "dV"), got, orc.attn_bwd(w.q, w.k, w.v, w.dout, w.offsets, **oracle_args(w))):
        check(what, g, r, TOL[dtype])
    check("dtable", to_np(dw.dtable), orc.attn_bwd_bias(w.q, w.k, w.v, w.dout, w.offsets, **oracle_args(w)), TOL[dtype])
