"""One workspace for the largest batch serves every smaller one: the sizes that the layer's queries give never fall as the token count grows, so that a
workspace sized for T tokens takes any T' <= T (with the room for dS where it had been asked for).  The backward in such a workspace returns what it
returns in one of its own size, bit for bit."""
import ctypes

import pytest

# (embed_dim, heads, head_dim): weight gradients of 4 to 512 output tiles, widths that are no multiples of 128 among them
WIDTHS = [(512, 2, 128), (128, 1, 128), (512, 4, 128), (256, 2, 64), (1024, 8, 128), (384, 6, 64), (72, 3, 64), (2048, 8, 128)]


@pytest.mark.parametrize("E,H,d", WIDTHS)
def test_layer_workspace_never_shrinks_with_more_tokens(E, H, d):
    from paper_2602_16986_amd import binding as hb
    lp = hb.HstuLayerParams()
    p = lp.attn
    p.batch, p.num_heads, p.head_dim, p.max_seqlen, p.dtype = 32, H, d, 2048, 0
    p.seq_offsets = 256                                                  # (never dereferenced by the size query)
    p.local_window, p.alpha, p.inv_n, lp.embed_dim = -1, 1.0, 1.0, E
    for query in (hb._lib.hstu_layer_workspace_bytes, hb._lib.hstu_layer_workspace_least_bytes):
        for backward in (0, 1):
            last = 0
            for T in sorted({1, 2, 63, 1792, 1793, *range(64, 40001, 64), *range(65, 40001, 640)}):
                p.total_tokens = T
                size = query(ctypes.byref(lp), backward)
                assert size >= last > 0 or last == 0 < size, f"{T} tokens take {size} bytes, fewer took {last}"
                last = size


@pytest.mark.gpu
@pytest.mark.parametrize("tokens,most,H,d,E", [(1792, 1793, 4, 128, 512), (4096, 4160, 2, 128, 512), (130, 8000, 1, 128, 128)])
def test_backward_in_a_workspace_sized_for_more_tokens(tokens, most, H, d, E):
    import torch
    from paper_2602_16986_amd import binding as hb
    from paper_2602_16986_amd import workloads as wl
    from paper_2602_16986_amd.runner import DeviceLayer
    lengths = lambda T: [128] * (T // 128) + ([T % 128] if T % 128 else [])
    dl = DeviceLayer(wl.build_layer("sizes", lengths(tokens), H, d, E, seed=1))
    dl.fwd()
    results = []
    outputs = ("dz", "d_norm_w", "d_w1", "d_gated_norm_w", "d_w2")
    dl.problem.params.attn.batch = len(lengths(most))
    dl.problem.params.attn.total_tokens = most
    sizes = [query(ctypes.byref(dl.problem.params), 1) for query in (hb._lib.hstu_layer_workspace_least_bytes, hb._lib.hstu_layer_workspace_bytes)]
    dl.problem.params.attn.batch = len(lengths(tokens))
    dl.problem.params.attn.total_tokens = tokens
    for size in (dl.ws_bwd.numel(), *sizes):
        dl.ws_bwd = hb.new_workspace(size, "cuda")
        for t in outputs:
            getattr(dl, t).fill_(float("nan"))
        dl.bwd()
        torch.cuda.synchronize()
        results.append([getattr(dl, t).clone() for t in outputs])
        assert all(torch.isfinite(t.float()).all() for t in results[-1])
    for a, b in zip(results[0], results[2]):                             # (the least size has no room for dS: another order of sums)
        assert torch.equal(a, b)
