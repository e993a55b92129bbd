"""Calls whose host copy of the offsets is not what the device holds: the lists are made on the device, the room for dS and the launches are
planned from the host's copy, and the two must not leave sums of memory that nobody wrote."""
import numpy as np
import pytest
import torch

from oracle import hstu_oracle as orc
from paper_2602_16986_amd import binding as hb
from paper_2602_16986_amd import workloads as wl
from test_gpu_parity import check, oracle_args, to_np, TOL

pytestmark = pytest.mark.gpu


def offsets_of(lengths):
    return np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)


@pytest.mark.parametrize("host,device", [([2048, 2048], [4096, 0]), ([3000, 1096], [4096, 0]), ([1500, 1500, 1096], [0, 4096, 0])])
def test_too_little_room_for_ds_leaves_every_output_untouched(host, device):
    """Host lengths whose blocks may be cut, so that the finishing launch runs; the device's need more room for dS."""
    T = sum(host)
    q = torch.randn(T, 1, 128, device="cuda").to(torch.bfloat16)
    outs = [torch.full_like(q, 5.0) for _ in range(3)]
    prob = hb.AttnProblem(q, q, q, q, torch.from_numpy(offsets_of(device)).cuda(), max_seqlen=T, seq_offsets_host=offsets_of(host))
    ws = hb.new_workspace(hb.hstu_attn_workspace_bytes(prob, True), "cuda")
    ws.fill_(0xFF)
    hb.hstu_attn_bwd(prob, q, q, q, q, *outs, ws)
    torch.cuda.synchronize()
    assert all(torch.all(t == 5.0) for t in outs)
    with pytest.raises(hb.HstuError) as e:
        hb.hstu_attn_schedule_stats(prob, ws, True)
    assert e.value.status == -2


@pytest.mark.parametrize("dim,dtype", [(128, "bf16"), (64, "bf16"), (32, "fp32")])
def test_longer_blocks_than_the_host_copy_has(dim, dtype):
    """Host lengths that leave nothing to cut, so that no launch finishes cut blocks, and device lengths whose blocks would be cut: the rows
    of every block are written."""
    from paper_2602_16986_amd.runner import DeviceWorkload
    w = wl.build("copy", [4096] + 15 * [0], 1, dim, dtype, seed=5, backward=True)
    dw = DeviceWorkload(w)
    prob = hb.AttnProblem(dw.q, dw.k, dw.v, dw.out, dw.offsets, max_seqlen=w.max_seqlen, seq_offsets_host=offsets_of(16 * [256]),
                          alpha=w.alpha, inv_n=1.0 / w.N, rab_table=dw.table, rab_bounds=dw.bounds)
    outs = [torch.full_like(dw.q, float("nan")) for _ in range(4)]
    hb.hstu_attn_fwd(prob, dw.q, dw.k, dw.v, outs[0], hb.new_workspace(hb.hstu_attn_workspace_bytes(prob, False), "cuda"))
    ws = hb.new_workspace(hb.hstu_attn_workspace_bytes(prob, True) - (256 if dim == 128 else 0), "cuda")     # (without room for dS)
    hb.hstu_attn_bwd(prob, dw.q, dw.k, dw.v, dw.dout, *outs[1:], ws)
    torch.cuda.synchronize()
    refs = [orc.attn_fwd(w.q, w.k, w.v, w.offsets, **oracle_args(w)), *orc.attn_bwd(w.q, w.k, w.v, w.dout, w.offsets, **oracle_args(w))]
    for what, got, ref in zip(("A", "dQ", "dK", "dV"), outs, refs):
        check(what, to_np(got), ref, TOL[dtype])
