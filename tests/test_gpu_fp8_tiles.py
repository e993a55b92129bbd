"""The FP8 product at the edges of its tiles and of the rule that chooses them: row counts beside whole tiles, columns that are no multiple of a tile's,
both reductions that take the pipelined tiles, and sizes for each of them and for the kernel with resident rows.  Against the product of the decoded
codes in float64.  Bound per element: half a step of bf16 (8 significant bits: 2^-8 of the value) and 2^-13 of the sum of the terms' magnitudes
for the matrix instruction's own sums of 64 products, which keep fewer bits than an fp32 sum: the kernel with resident rows shows up to
4.9e-5 of it (K = 256), the tiles 2.7e-5 (K = 1024); a first bound of K 2^-24 took them for fp32 sums.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 64, 512), (63, 192, 1024), (65, 320, 512), (129, 64, 1024), (193, 576, 1024), (257, 192, 512), (300, 64, 256),
                                   (2001, 2048, 1024), (4099, 2048, 512), (6001, 1024, 1024), (16385, 128, 512)])
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
    rows = torch.unique(torch.cat([torch.arange(min(M, 300)), torch.arange(max(M - 300, 0), M)]))
    dec = lambda t: t.cpu().view(torch.float8_e4m3fn).double()
    x, w = dec(a[rows.cuda()]), dec(b)
    scale = sa.cpu().double()[rows][:, None] * sb.cpu().double()[None]
    ref, size = (x @ w.T) * scale, (x.abs() @ w.abs().T) * scale
    if residual:
        ref += c[rows.cuda()].cpu().double()
    err = (d[rows.cuda()].cpu().double() - ref).abs()
    assert (err <= 2.0 ** -8 * ref.abs() + 2.0 ** -13 * size).all(), float((err / (ref.abs() + size)).max())
    assert torch.isnan(d[M:].float()).all(), "rows past the end written"
