"""The products over token rows inside the layer, at the edges of their tiles: token counts just beside and beyond whole tiles, widths that
are no multiple of a tile's columns or of a k-tile, and a size for every tile the size rule knows (with 2048 projection columns: 64 rows up to
about 2,000 tokens, 128 rows in both depths, 192 and 256 rows).  Forward and every gradient against the fp64 layer oracle."""
import pytest
import torch

from paper_2602_16986_amd import workloads as wl
from test_gpu_layer import hb, run_case  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,d,E", [
    (1, 1, 32, 8),            # one row, one k-tile of 8
    (63, 1, 64, 72), (65, 3, 64, 328), (129, 1, 32, 136), (255, 5, 64, 200), (257, 2, 128, 1032),
    (1990, 4, 128, 64), (2049, 4, 128, 136), (4161, 4, 128, 72), (6401, 4, 128, 136),
    # weight gradients of widths that are multiples of 128: one slab of token rows, ragged slabs, more tiles than compute units
    (7, 1, 128, 128), (130, 2, 128, 384), (1601, 4, 128, 512), (5003, 1, 128, 256), (200, 9, 128, 1152)])
def test_layer_products_at_tile_edges(hb, T, H, d, E):
    lengths = [60] * (T // 60) + ([T % 60] if T % 60 else [])
    run_case(wl.build_layer(f"products-{T}-{H}-{d}-{E}", lengths, H, d, E, seed=T + E, K1=40, K2=8))


def test_rows_do_not_touch_each_other(hb):
    """A token row that is not finite stays in its own row of the projections: U of every other row is what it was."""
    from paper_2602_16986_amd.runner import DeviceLayer
    dl = DeviceLayer(wl.build_layer("rows", [60, 33, 40], 2, 64, 72, seed=5))
    dl.fwd()
    before = dl.u_saved.clone()
    dl.z[70] = float("nan")
    dl.fwd()
    torch.cuda.synchronize()
    keep = torch.arange(before.shape[0], device=before.device) != 70
    assert torch.equal(dl.u_saved[keep], before[keep])
    assert torch.isnan(dl.u_saved[70].float()).all()
