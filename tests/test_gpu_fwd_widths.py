"""The pipelined forward at every width: rows of 64, 128 and 256 bytes have their own LDS layout and loads per wave.  Sequence lengths at the edges of its
32-key sub-blocks and 128-row blocks, a prefix that is not a multiple of 32, candidates, a query tail, and blocks cut along the key
axis, against the oracle.  Tolerance 2e-2 (bf16 storage) as in test_gpu_parity.py."""
import numpy as np
import pytest
import torch

from oracle import hstu_oracle as orc
from paper_2602_16986_amd import workloads as wl
from test_gpu_parity import check, oracle_args, to_np, TOL

pytestmark = pytest.mark.gpu

CASES = {                               # lengths, K1, K2, candidates, query tail
    "edges": ([1, 2, 31, 32, 33, 64, 95, 127, 128, 129, 160, 257], -1, 0, None, 0),
    "band": ([300, 33, 129, 511], 70, 45, None, 0),
    "candidates": ([333, 97, 128, 260], 100, 17, [40, 97, 0, 132], 0),
    "tail": ([900, 40, 257], -1, 0, [33, 0, 5], 50),
    "cut": ([2500], -1, 0, None, 0),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("d", [32, 64, 128])
def test_forward(d, name):
    from paper_2602_16986_amd.runner import DeviceWorkload
    lengths, K1, K2, targets, tail = CASES[name]
    w = wl.build(name, lengths, 2, d, "bf16", seed=5, K1=K1, K2=K2, num_targets=None if targets is None else np.array(targets, dtype=np.int32))
    dw = DeviceWorkload(w)
    dw.problem.params.query_tail = tail
    dw.out.fill_(7.0)
    dw.ws_fwd.fill_(0xFF)
    got = to_np(dw.attn_fwd())
    torch.cuda.synchronize()
    ref = orc.attn_fwd(w.q, w.k, w.v, w.offsets, **oracle_args(w))
    rows = np.ones(w.T, dtype=bool)
    if tail:
        for b, (o, e) in enumerate(zip(w.offsets[:-1], w.offsets[1:])):
            rows[o:max(int(e) - int(targets[b]) - tail, int(o))] = False
        assert np.all(got[~rows] == 7.0)
    check("A", got[rows], ref[rows], TOL["bf16"])
