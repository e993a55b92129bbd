"""Bias strips of the streamed tiles, all widths and types: what lies around the rows of the expanded bias table may be
fetched with a strip, so no output may show it (the workspaces hold NaN wherever nothing was written).  Tolerances as in
test_gpu_parity.py: 2e-2 for bf16 storage, 1e-5 for fp32."""
import numpy as np
import pytest
import torch

from oracle import hstu_oracle as orc
from paper_2602_16986_amd import workloads as wl
from test_gpu_parity import check, oracle_args, to_np, TOL

pytestmark = pytest.mark.gpu

MASKS = {"dense": (-1, 0, None), "window": (40, 20, None), "window-candidates": (70, 0, [0, 1, 5, 32, 33, 40, 129, 60, 90])}


@pytest.mark.parametrize("mask", list(MASKS))
@pytest.mark.parametrize("dtype,d", [("bf16", 32), ("bf16", 64), ("bf16", 128), ("fp32", 32), ("fp32", 128)])
def test_forward_and_backward_in_nan_workspaces(dtype, d, mask):
    from paper_2602_16986_amd.runner import DeviceWorkload
    K1, K2, targets = MASKS[mask]
    w = wl.build("strip", [1, 31, 32, 33, 127, 128, 129, 161, 290], 3, d, dtype, seed=11, K1=K1, K2=K2, backward=True,
                 num_targets=None if targets is None else np.array(targets, dtype=np.int32))
    dw = DeviceWorkload(w)
    for t in (dw.ws_fwd, dw.ws_bwd):
        t.fill_(0xFF)
    for t in (dw.out, dw.dq, dw.dk, dw.dv):
        t.fill_(float("nan"))
    dw.attn_fwd()
    dw.attn_bwd()
    torch.cuda.synchronize()
    check("A", to_np(dw.out), orc.attn_fwd(w.q, w.k, w.v, w.offsets, **oracle_args(w)), TOL[dtype])
    refs = orc.attn_bwd(w.q, w.k, w.v, w.dout, w.offsets, **oracle_args(w))
    for what, g, r in zip(("dQ", "dK", "dV"), (dw.dq, dw.dk, dw.dv), refs):
        check(what, to_np(g), r, TOL[dtype])
