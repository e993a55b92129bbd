"""Truncation of narrow rows, of which one instruction moves one or several by a rule on their number: row widths that do and do not divide a wave's lanes,
batches whose steps cross one, a few, or more sequences than a wave holds at a time, empty ones among them, on both sides of the rule.  Bit for bit against the numpy oracle, both directions."""
import numpy as np
import pytest
import torch

from oracle import truncation as orc

pytestmark = pytest.mark.gpu

BATCHES = {
    "one": lambda rng: np.array([1000]),
    "ordinary": lambda rng: rng.integers(0, 300, size=70),
    "tiny": lambda rng: rng.integers(0, 3, size=5000),
    "mostly empty": lambda rng: np.where(rng.random(900) < 0.9, 0, rng.integers(1, 40, size=900)),
    "long": lambda rng: np.array([9000, 3]),
    "many tiny": lambda rng: rng.integers(0, 3, size=70000),
    "many mostly empty": lambda rng: np.where(rng.random(50000) < 0.9, 0, rng.integers(1, 40, size=50000)),
    "empty ends": lambda rng: np.concatenate([np.zeros(130, int), [77, 0, 5], np.zeros(100, int)]),
}


@pytest.mark.parametrize("batch", BATCHES)
@pytest.mark.parametrize("row_bytes", [16, 48, 176, 512, 528])
@pytest.mark.parametrize("targets", [False, True])
def test_truncation_of_narrow_rows(batch, row_bytes, targets):
    from paper_2602_16986_amd import binding as hb
    rng = np.random.default_rng(row_bytes)
    lengths = BATCHES[batch](rng).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    nt = np.minimum(rng.integers(0, 4, size=len(lengths)), lengths).astype(np.int32) if targets else None
    keep, width, T = 9, row_bytes // 2, int(off[-1])
    x = rng.integers(-30000, 30000, size=(T, width), dtype=np.int16)
    ref, ref_off = orc.tail_slice(x, off, keep, nt)
    dev = torch.device("cuda:0")
    d_off, d_nt, d_x = torch.from_numpy(off).to(dev), None if nt is None else torch.from_numpy(nt).to(dev), torch.from_numpy(x).to(dev)
    d_new = torch.empty(len(off), dtype=torch.int32, device=dev)
    y = torch.full((len(ref) + 3, width), 0x5A5A, dtype=torch.int16, device=dev)
    hb.hstu_truncate_offsets(d_off, keep, d_nt, d_new)
    hb.hstu_truncate_fwd(d_off, d_new, d_x, y)
    dy = rng.integers(-30000, 30000, size=ref.shape, dtype=np.int16)
    dx = torch.full((T, width), 0x5A5A, dtype=torch.int16, device=dev)
    hb.hstu_truncate_bwd(d_off, d_new, torch.from_numpy(dy).to(dev), dx)
    torch.cuda.synchronize()
    assert np.array_equal(d_new.cpu().numpy(), ref_off)
    assert np.array_equal(y[:len(ref)].cpu().numpy(), ref)
    assert (y[len(ref):] == 0x5A5A).all(), "rows past the end written"
    assert np.array_equal(dx.cpu().numpy(), orc.tail_slice_bwd(dy, off, keep, nt))
