"""The pipelined backward for 32 and 64 features: edges of its 32-row tiles and 128-row blocks, key blocks that hold the end of a global prefix, candidates,
blocks cut into pieces, the table's gradient, in workspaces full of NaN, against the oracle.  Tolerance 2e-2 (bf16 storage) as in
test_gpu_parity.py."""
import numpy as np
import pytest
import torch

from oracle import hstu_oracle as orc
from paper_2602_16986_amd import workloads as wl
from test_gpu_parity import check, oracle_args, to_np, TOL

pytestmark = pytest.mark.gpu

CASES = {                               # lengths, K1, K2, candidates
    "edges": ([1, 2, 31, 32, 33, 64, 95, 127, 128, 129, 160, 257], -1, 0, None),
    "window-below-a-tile": ([300, 129, 1], 5, 0, None),
    "prefix-inside-a-block": ([700, 513, 90], 130, 70, None),
    "prefix-of-whole-blocks": ([700, 513, 90], 130, 256, None),
    "prefix-only": ([400, 300], 0, 100, None),
    "prefix-only-candidates": ([400, 300, 131], 0, 100, [90, 0, 131]),
    "candidates": ([333, 97, 128, 260], -1, 0, [40, 97, 0, 132]),
    "window-candidates": ([600, 340, 97], 64, 33, [250, 31, 1]),
    "cut": ([2600], -1, 0, None),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("d", [32, 64])
def test_backward(d, name):
    from paper_2602_16986_amd.runner import DeviceWorkload
    lengths, K1, K2, targets = CASES[name]
    w = wl.build(name, lengths, 2, d, "bf16", seed=9, K1=K1, K2=K2, backward=True,
                 num_targets=None if targets is None else np.array(targets, dtype=np.int32))
    refs = orc.attn_bwd(w.q, w.k, w.v, w.dout, w.offsets, **oracle_args(w))
    ref_table = orc.attn_bwd_bias(w.q, w.k, w.v, w.dout, w.offsets, **oracle_args(w))
    for bias_grad in (False, True):
        dw = DeviceWorkload(w, bias_grad=bias_grad)
        dw.ws_bwd.fill_(0xFF)
        for t in (dw.dq, dw.dk, dw.dv):
            t.fill_(float("nan"))
        dw.attn_bwd()
        torch.cuda.synchronize()
        for what, g, r in zip(("dQ", "dK", "dV"), (dw.dq, dw.dk, dw.dv), refs):
            check(what, to_np(g), r, TOL["bf16"])
        if bias_grad:
            check("dtable", to_np(dw.dtable), ref_table, TOL["bf16"])
