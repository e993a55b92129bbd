"""The products over token rows inside the layer, at the edges of their tiles: token counts just beside and beyond whole tiles, widths that are no
multiple of a tile's columns or of a k-tile, and sizes for every tile that the size rule knows, in each of the products, with workgroups that go
through several tiles and without (test_sizes_reach_every_tile asks the rule itself).  Forward and every gradient against the fp64 layer oracle."""
import ctypes
import os
import subprocess

import pytest
import torch

from paper_2602_16986_amd import workloads as wl
from test_gpu_layer import hb, run_case  # noqa: F401

CASES = [
    (1, 1, 32, 8),            # one row, one k-tile of 8
    (63, 1, 64, 72), (65, 3, 64, 328), (129, 1, 32, 136), (255, 5, 64, 200), (257, 2, 128, 1032),
    (1990, 4, 128, 64), (2049, 4, 128, 136), (4161, 4, 128, 72), (6401, 4, 128, 136),
    # weight gradients of widths that are multiples of 128: one slab of token rows, ragged slabs, more tiles than compute units
    (7, 1, 128, 128), (130, 2, 128, 384), (1601, 4, 128, 512), (5003, 1, 128, 256), (200, 9, 128, 1152),
    # the tiles that the sizes above leave out
    (150, 36, 128, 64), (570, 1, 128, 7000), (3300, 5, 32, 64), (8200, 4, 128, 64), (8200, 3, 128, 64), (8200, 5, 32, 136), (10300, 4, 128, 64),
    (10300, 13, 128, 64), (12900, 13, 128, 64), (6401, 8, 128, 64), (6401, 36, 128, 64), (5000, 13, 128, 64), (12900, 8, 128, 64), (12900, 1, 128, 264), (14500, 1, 128, 520), (12900, 1, 128, 776), (5000, 1, 128, 4104), (25000, 8, 128, 1000)]


@pytest.mark.gpu
@pytest.mark.parametrize("T,H,d,E", CASES)
def test_layer_products_at_tile_edges(hb, T, H, d, E):
    lengths = [60] * (T // 60) + ([T % 60] if T % 60 else [])
    run_case(wl.build_layer(f"products-{T}-{H}-{d}-{E}", lengths, H, d, E, seed=T + E, K1=40, K2=8))


@pytest.fixture(scope="module")
def product_tile(tmp_path_factory):
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_16986_amd", "csrc")
    so = str(tmp_path_factory.mktemp("tiles") / "libtiles.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(csrc, "geometry_check.cpp")])
    lib = ctypes.CDLL(so)
    lib.product_tile.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    return lib.product_tile


TILES = {1: (64, 128, 256), 2: (64, 128, 512), 3: (128, 128, 256), 4: (128, 128, 512), 5: (192, 256, 256), 6: (256, 256, 256)}   # rows, columns, workgroups


def reached(products, tile_of, tiles):
    """{(product, tile, whether workgroups go through several tiles)}"""
    got = set()
    for name, M, N, K in products:
        t = tile_of(M, N, K, name)
        rows, cols, workgroups = tiles[t]
        got.add((name, t, -(-M // rows) * -(-N // cols) > workgroups))
    return got


def test_sizes_reach_every_tile(product_tile):
    """U/V/Q/K (both epilogues), the output with its residual, and the products with W [K, N].  64-row tiles go through several per workgroup nowhere, and
    256-row tiles take a residual with long reductions only (which the largest size has)."""
    products = []
    for T, H, d, E in CASES:
        HD = H * d
        products += [("uvqk", T, 4 * HD, E), ("out", T, E, HD), ("nn", T, HD, E), ("nn", T, E, 4 * HD)]
    got = reached(products, lambda M, N, K, name: product_tile(M, N, K, name == "out", 0), TILES)
    several = {(t, s) for t in (4, 5, 6) for s in (False, True)} | {(1, False), (2, False), (3, False)}
    missing = {(name, t, s) for name in ("uvqk", "out", "nn") for t, s in several} - got
    assert missing <= {("out", 6, False)}, missing


@pytest.mark.gpu
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
