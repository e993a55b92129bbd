"""The FP8 product at the edges of its tiles and of the rule that chooses them: row counts beside whole tiles, columns that are no multiple of a tile's,
both reductions that take the pipelined tiles, and sizes for each of them, with workgroups that go through several tiles and without
(test_sizes_reach_every_tile asks the rule itself), and for the kernel with resident rows.  Against the product of the decoded
codes in float64.  Bound per element: half a step of bf16 (8 significant bits: 2^-8 of the value) and 2^-13 of the sum of the terms' magnitudes
for the matrix instruction's own sums of 64 products, which keep fewer bits than an fp32 sum: the kernel with resident rows shows up to
4.9e-5 of it (K = 256), the tiles 2.7e-5 (K = 1024); a first bound of K 2^-24 took them for fp32 sums.
"""
import pytest
import torch

from paper_2602_16986_amd import workloads as wl
from test_gpu_layer import attn_kw, check, f64, lorc
from test_gpu_layer_products import product_tile, reached  # noqa: F401

CASES = [(1, 64, 512), (63, 192, 1024), (65, 320, 512), (129, 64, 1024), (193, 576, 1024), (257, 192, 512), (300, 64, 256),
         (2001, 2048, 1024), (4099, 2048, 512), (6001, 1024, 1024), (16385, 128, 512),
         (129, 64, 512), (12001, 576, 512), (12001, 320, 512), (14001, 1024, 512), (14001, 576, 512), (5000, 4032, 512), (6001, 1984, 512)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", CASES)
@pytest.mark.parametrize("residual", [False, True])
def test_fp8_product_at_tile_edges(M, N, K, residual):
    from paper_2602_16986_amd import binding as hb
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    codes = lambda r: (torch.randint(0, 0x70, (r, K), generator=gen, device="cuda") + 0x80 * torch.randint(0, 2, (r, K), generator=gen, device="cuda")).to(torch.uint8)
    a, b = codes(M), codes(N)
    sa, sb = (torch.rand(n, generator=gen, device="cuda") * 0.01 + 0.001 for n in (M, N))
    c = torch.randn(M, N, generator=gen, device="cuda").to(torch.bfloat16) if residual else None
    d = torch.full((M + 256, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    hb.hstu_fp8_gemm_bias2d(a, sa, b, sb, c, d[:M])
    torch.cuda.synchronize()
    rows = torch.unique(torch.cat([torch.arange(min(M, 300)), torch.arange(0, M, 29), torch.arange(max(M - 300, 0), M)]))     # (some of every row tile)
    dec = lambda t: t.cpu().view(torch.float8_e4m3fn).double()
    x, w = dec(a[rows.cuda()]), dec(b)
    scale = sa.cpu().double()[rows][:, None] * sb.cpu().double()[None]
    ref, size = (x @ w.T) * scale, (x.abs() @ w.abs().T) * scale
    if residual:
        ref += c[rows.cuda()].cpu().double()
    err = (d[rows.cuda()].cpu().double() - ref).abs()
    assert (err <= 2.0 ** -8 * ref.abs() + 2.0 ** -13 * size).all(), float((err / (ref.abs() + size)).max())
    assert torch.isnan(d[M:].float()).all(), "rows past the end written"


LAYERS = [(200, 1, 512), (4099, 1, 512), (4099, 8, 512), (4099, 2, 512), (14001, 2, 512), (4099, 4, 512), (5000, 8, 512)]     # tokens, heads of 128, embed_dim


@pytest.mark.gpu
@pytest.mark.parametrize("T,H,E", LAYERS)
def test_fp8_projection_with_silu_at_tile_edges(T, H, E):
    """The epilogue with SiLU and the gate's columns apart, through the layer's forward, against its oracle with the bounds of test_layer_forward_fp8."""
    from paper_2602_16986_amd.runner import DeviceLayer
    c = wl.build_layer(f"fp8-tiles-{T}", [60] * (T // 60) + [T % 60], H, 128, E, seed=T, K1=20)
    dl = DeviceLayer(c, fp8=True)
    for t in (dl.out, dl.u_saved, dl.attn_saved):
        t.fill_(float("nan"))
    dl.fwd()
    torch.cuda.synchronize()
    ref, s = lorc.layer_fwd_fp8(c.z, c.norm_w, c.w1, c.gated_norm_w, c.w2, c.offsets, c.H, c.d, norm_eps=c.eps, gated_eps=c.eps, **attn_kw(c))
    check("U (saved)", f64(dl.u_saved), s["u"], 5e-2, 4e-3)
    check("A (saved)", f64(dl.attn_saved), s["a"], 5e-2, 4e-3)
    check("out", f64(dl.out), ref, 5e-2, 4e-3)


def test_sizes_reach_every_tile(product_tile):
    tiles = {1: (64, 128, 256), 2: (64, 128, 512), 4: (128, 256, 256), 5: (192, 256, 256)}                    # rows, columns, workgroups
    tiled = lambda M, K: M > 40 if K == 1024 else K == 512 and 80 < M <= 16384                              # (fp8_gemm.hip: the others have a kernel of their own)
    products = [(name, M, N, K) for name in ("plain", "residual") for M, N, K in CASES if tiled(M, K)]
    products += [("silu", T, 4 * 128 * H, E) for T, H, E in LAYERS if tiled(T, E)]
    got = reached(products, lambda M, N, K, name: product_tile(M, N, K, name == "residual", 1), tiles)
    several = {(1, False)} | {(t, s) for t in (2, 4, 5) for s in (False, True)}
    assert got == {(name, t, s) for name in ("plain", "silu", "residual") for t, s in several if name != "residual" or t != 5}
