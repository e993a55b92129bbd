"""What a token row gets from the FP8 products does not depend on how many rows are beside it, though the kernel and its tiles do: bit for bit, on both sides
of every line of the rules that choose them."""
import pytest
import torch

from paper_2602_16986_amd import binding as hb
from paper_2602_16986_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [(128, 512), (1024, 512), (192, 1024), (1024, 1024)])
@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("codes", ["quantised", "uniform"])
def test_fp8_product_rows_do_not_depend_on_the_row_count(N, K, residual, codes):
    most = 20600
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    quantised = lambda t: (torch.empty(t.shape, dtype=torch.uint8, device="cuda"), torch.empty(t.shape[0], device="cuda"))
    (a, sa), (b, sb) = (quantised(t) for t in (torch.empty(most, K), torch.empty(N, K)))
    for q, s in ((a, sa), (b, sb)):
        hb.hstu_norm_quant_fp8(torch.randn(q.shape, generator=gen, device="cuda").bfloat16(), None, None, None, 0.0, q, s)
        if codes == "uniform":                               # every exponent as often as any other: sums of very unequal terms
            q.copy_(torch.randint(0, 0x7F, q.shape, generator=gen, device="cuda") + 0x80 * torch.randint(0, 2, q.shape, generator=gen, device="cuda"))
    c = torch.randn(most, N, generator=gen, device="cuda").bfloat16() if residual else None
    got = []
    for rows in (most, 16385, 16384, 5000, 300, 129, 81, 80, 65, 41, 40, 1):
        d = torch.empty(rows, N, dtype=torch.bfloat16, device="cuda")
        hb.hstu_fp8_gemm_bias2d(a[:rows], sa[:rows], b, sb, c[:rows] if residual else None, d)
        got.append(d)
    torch.cuda.synchronize()
    for d in got[1:]:
        assert torch.equal(d, got[0][:len(d)]), f"{len(d)} rows: {int((d != got[0][:len(d)]).sum())} elements differ"


@pytest.mark.parametrize("E", [512, 1024])
def test_fp8_layer_rows_do_not_depend_on_the_token_count(E):
    """The first projection with its SiLU, through the layer: the saved gate of the first tokens, in batches of 20,000 and fewer."""
    from paper_2602_16986_amd.runner import DeviceLayer
    layer = lambda n: DeviceLayer(wl.build_layer("rows", [20] * n, 2, 128, E, seed=3, K1=16), fp8=True)
    whole = layer(1000)
    whole.fwd()
    for n in (815, 100, 5, 4, 3, 2, 1):
        part = layer(n)
        for t in ("z", "w1_q", "w1_scale", "norm_w"):
            getattr(part, t).copy_(getattr(whole, t)[:getattr(part, t).shape[0]])
        part.fwd()
        torch.cuda.synchronize()
        assert torch.equal(part.u_saved, whole.u_saved[:20 * n]), n
