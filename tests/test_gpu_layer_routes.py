"""Layer products on both sides of the line between this library's own kernels and the GEMM library.  The line goes by the shape class of the token count
(rounded up to a power of two), so that a call of a class decides the route, and makes the choice of the library's kernels, for every call of it."""
import pytest
import torch

from paper_2602_16986_amd import workloads as wl
from test_gpu_layer import hb, run_case  # noqa: F401

pytestmark = pytest.mark.gpu


def lengths(T):
    return [64] * (T // 64) + ([T % 64] if T % 64 else [])


@pytest.mark.parametrize("T,same_class,H,E", [(16500, 32000, 8, 1024), (33000, 60000, 8, 1024), (66000, 100000, 4, 512)])
def test_one_call_of_a_class_leaves_nothing_to_tune(hb, T, same_class, H, E):
    """A forward and a backward at one token count, then others of the same class above it and below: none of them times candidates."""
    from paper_2602_16986_amd.runner import DeviceLayer
    layer = lambda n: DeviceLayer(wl.build_layer("route", lengths(n), H, 128, E, seed=n, K1=32))
    layer(T).step()
    tuned = hb.hstu_layer_gemm_tunings()
    for n in (same_class, (1 << (T - 1).bit_length()), (1 << ((T - 1).bit_length() - 1)) + 1):
        dl = layer(n)
        dl.step()
        torch.cuda.synchronize()
        assert hb.hstu_layer_gemm_tunings() == tuned, f"{n} tokens, after {T}"
        assert torch.isfinite(dl.dz.float()).all() and torch.isfinite(dl.out.float()).all()


@pytest.mark.parametrize("T,products", [(2048, (0, 0)), (2100, (2, 2)), (8193, (3, 3))])
def test_products_of_the_library_against_the_oracle(hb, T, products):
    """E = 8192, H d = 2048: no product of the class of 2,048 tokens takes 10^11 multiply-adds at half of them, the projection (twice, for the gate's columns
    apart) and its input gradient of the class of 4,096 do, and all of the class of 16,384.  How many new products were tuned, forward and backward, says that they ran there."""
    from paper_2602_16986_amd.runner import DeviceLayer
    c = wl.build_layer(f"route-{T}", lengths(T), 16, 128, 8192, seed=T, K1=40, K2=8)
    dl, tuned = DeviceLayer(c), [hb.hstu_layer_gemm_tunings()]
    for call in (dl.fwd, dl.bwd):
        call()
        torch.cuda.synchronize()
        tuned.append(hb.hstu_layer_gemm_tunings())
    assert (tuned[1] - tuned[0], tuned[2] - tuned[1]) == products
    run_case(c)


def test_layer_step_with_products_of_the_library_replays_from_a_graph(hb):
    from paper_2602_16986_amd.runner import DeviceLayer
    from test_gpu_graph_capture import _capture_and_replay
    dl = DeviceLayer(wl.build_layer("route-graph", lengths(2200), 16, 128, 8192, seed=1, K1=40, K2=8))
    dl.step()
    tuned = hb.hstu_layer_gemm_tunings()
    _capture_and_replay(dl.step, [dl.out, dl.dz, dl.d_norm_w, dl.d_w1, dl.d_gated_norm_w, dl.d_w2], dl.device)
    assert hb.hstu_layer_gemm_tunings() == tuned
