"""Group-128 scales on one to two rounds of 128x256 tiles: every tile in two pieces at the same stage,
the second to end adding the first one's sums.  Against the CPU oracle at the edges (two stages, one
tile, rows and columns that end inside one, several pieces a workgroup), and the library's own choice."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_04405_amd as fq
from paper_2508_04405_amd import dev, synth

from gpu_helpers import assert_y_close, group_slack, say, to_dev
from test_gpu_group_order import call, check_scales_that_are_not_finite, operands
from test_gpu_xgroup import assert_close, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("both,bits", [(False, 6), (True, 8)])
@pytest.mark.parametrize("M,K,N", [(1, 256, 32), (129, 384, 544), (300, 640, 288), (1029, 256, 7456), (1025, 896, 7712)])
def test_pairs(M, K, N, both, bits):
    say(f"group pairs M={M} K={K} N={N} both={both} A{bits}")
    w, x16, packed, codes = operands(M, K, N, both, bits)
    tiles = (M + 127) // 128 * ((N + 255) // 256)
    ws = fq.make_workspace(M, N, K, extra=tiles << 18)
    dev.set_dispatch(2, 0, 0, 22)
    try:
        out = [call(packed, N, K, codes, both, bits, ws) for _ in range(3)]
        assert dev.last_dispatch()[0] == 22
    finally:
        dev.set_dispatch()
    assert int(ws[:16384].view(torch.int32).abs().sum()) == 0
    # two fp32 sums have no order: whoever ends second, the bits are the same
    for o in out[1:]:
        assert np.array_equal(o.view(np.uint16), out[0].view(np.uint16))
    if both:
        _, _, ry, slack = reference(x16, w, bits)
        assert_close(out[0], ry, slack, "pairs:")
    else:
        ref = oracle.linear(x16, w, bits, 128)
        assert_y_close(out[0], ref["y"], group_slack(ref))


# the line: one to two rounds, 32 stages, and what the shorter round is worth; the workspace does not show
@pytest.mark.parametrize("both", [False, True])
@pytest.mark.parametrize("M,K,N,pairs", [(1100, 8192, 8192, True), (1100, 3968, 8192, False), (1024, 8192, 8192, False),
                                         (2048, 5120, 5120, False), (1700, 13824, 5120, True)])
def test_choice_and_equal_tokens(M, K, N, pairs, both):
    say(f"group pairs, the library's choice: M={M} K={K} N={N} both={both}")
    half = synth.activations(M // 2, K, seed=7, outlier_frac=0.02)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    packed = fq.pack_w6(*fq.quant_w6(torch.randn((N, K), generator=g, device="cuda") * 0.02, 128), 128)
    codes = (fq.quant_act_g128 if both else fq.quant_act)(to_dev(np.tile(half, (2, 1))), 8)
    exact, roomy = fq.make_workspace(M, N, K), fq.make_workspace(M, N, K, extra=64 << 20)
    y = call(packed, N, K, codes, both, 8, exact)
    assert (dev.last_dispatch()[0] == 22) == pairs
    assert np.array_equal(call(packed, N, K, codes, both, 8, roomy).view(np.uint16), y.view(np.uint16))
    assert np.array_equal(y[:M // 2].view(np.uint16), y[M // 2:].view(np.uint16))
    # one K split asked for: no form cuts K, and all that do not agree
    dev.set_dispatch(2, 1, 0, 18)
    try:
        whole = call(packed, N, K, codes, both, 8, exact)
        dev.set_dispatch(2, 1)
        forced = call(packed, N, K, codes, both, 8, exact)
        assert dev.last_dispatch() in ((18, 1), (19, 1))
    finally:
        dev.set_dispatch()
    assert np.array_equal(forced.view(np.uint16), whole.view(np.uint16))
    assert pairs or np.array_equal(y.view(np.uint16), whole.view(np.uint16))
    whole = whole.astype(np.float64)
    # the same terms in one chain and in two: fp32 sums of K / 128 terms, then one rounding to fp16.
    # Relative to the output's spread the chains differ by far less than fp16's 2^-11.
    d = np.abs(y.astype(np.float64) - whole)
    assert d.max() <= 2.0 ** -10 * np.abs(whole).max()
    assert np.linalg.norm(d) <= 2.0 ** -13 * np.linalg.norm(whole)


@pytest.mark.parametrize("both", [False, True])
def test_scales_that_are_not_finite(both):
    check_scales_that_are_not_finite(22, both)      # (infinities of both signs in different pieces among them)


def test_in_the_block_runner():
    """The output projection of a wide block takes the pairs: the bits of the layer called by itself."""
    M, H, F, QKV = 1052, 8192, 128, 32
    say("group pairs in the block runner")
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    packed = [fq.pack_w6(*fq.quant_w6(torch.randn(s, generator=g, device="cuda") * 0.02, 128), 128)
              for s in ((QKV, H), (H, H), (2 * F, H), (H, F))]
    gain = torch.ones(H, dtype=torch.float16, device="cuda")
    layer = fq.Layer(H, F, QKV, 128, *packed, gain, gain, 1e-5, (6, 6, 6, 8))
    attn = to_dev(synth.activations(M, H, seed=9, outlier_frac=0.02))
    o = torch.empty((M, H), dtype=torch.float16, device="cuda")
    alone = dev.gemm_w6a6(packed[1], H, H, 128, x_fp16=attn)
    assert dev.last_dispatch()[0] == 22
    ws = layer.make_workspace(M)
    for _ in range(2):
        fq.layer_linears(layer, M, ws, 1, 1, attn=attn, o=o)
        assert torch.equal(o, alone)
    assert int(ws[:16384].view(torch.int32).abs().sum()) == 0


def test_captured_and_replayed():
    M, K, N = 1029, 640, 7456
    say("group pairs, captured")
    _, _, packed, _ = operands(M, K, N, False)
    x = to_dev(synth.activations(M, K, seed=M))
    ws, y = fq.make_workspace(M, N, K, extra=128 << 20), torch.empty((M, N), dtype=torch.float16, device="cuda")
    dev.set_dispatch(2, 0, 0, 22)
    try:
        run = lambda: dev.gemm_w6a8(packed, N, K, 128, x_fp16=x, workspace=ws, out=y)
        run()
        torch.cuda.synchronize()
        stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.stream(stream):
            with torch.cuda.graph(graph, stream=stream):
                run()
        for rep in range(3):
            x.copy_(to_dev(synth.activations(M, K, seed=100 + rep)))
            graph.replay()
            torch.cuda.synchronize()
            got = y.clone()
            run()
            torch.cuda.synchronize()
            assert torch.equal(got, y), rep
    finally:
        dev.set_dispatch()
