"""Group-128 scales: the fp32 sums over the groups are taken in one order, whichever tiled kernel
runs.  The library's own choice gives the bits of the 128x128 tiles with the same K splits, for
every row of a call and with any workspace; the 64x256 tiles are compared with the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_04405_amd as fq
from paper_2508_04405_amd import dev, synth

from gpu_helpers import assert_y_close, group_slack, say, to_dev
from test_gpu_xgroup import assert_close, reference

pytestmark = pytest.mark.gpu


def operands(M, K, N, both, bits=8, x16=None):
    w = synth.weights(N, K, 0.02, seed=K + N)
    x16 = synth.activations(M, K, seed=M, outlier_frac=0.02) if x16 is None else x16
    packed = fq.pack_w6(*fq.quant_w6(to_dev(w), 128), 128)
    codes = (fq.quant_act_g128 if both else fq.quant_act)(to_dev(x16), bits)
    return w, x16, packed, codes


def call(packed, N, K, codes, both, bits, ws):
    if both:
        return dev.linear_g128(packed, N, K, *codes, workspace=ws).cpu().numpy()
    fn = dev.gemm_w6a6 if bits == 6 else dev.gemm_w6a8
    return fn(packed, N, K, 128, xq=codes[0], sx=codes[1], workspace=ws).cpu().numpy()


# want: the form and its K splits -- split or whole, at half the height or not, one round or
# several, a tail of one tile, columns and rows that end inside a tile
@pytest.mark.parametrize("both", [False, True])
@pytest.mark.parametrize("M,K,N,want", [
    (65, 4096, 5120, (8, 5)), (97, 8192, 8192, (19, 4)), (97, 2048, 16384, (19, 1)), (97, 8192, 10240, (19, 3)),
    (100, 1536, 40960, (18, 1)), (129, 2048, 4096, (19, 1)), (200, 4480, 1056, (19, 2)), (200, 16384, 8192, (18, 4)),
    (333, 1024, 13664, (18, 1)), (700, 4096, 5120, (19, 1)), (2048, 3200, 5120, (19, 1)), (1029, 256, 7456, (19, 1)),
    (33 * 128, 384, 1824, (19, 1))])
def test_same_bits_in_every_form(M, K, N, want, both):
    say(f"group order: M={M} K={K} N={N} both={both}")
    _, _, packed, codes = operands(M, K, N, both)
    exact = fq.make_workspace(M, N, K)
    roomy = fq.make_workspace(M, N, K, extra=64 << 20)
    y = call(packed, N, K, codes, both, 8, exact)
    launched = [dev.last_dispatch()]
    again = call(packed, N, K, codes, both, 8, roomy)
    launched.append(dev.last_dispatch())
    dev.set_dispatch(2, 0, 0, 8)
    try:
        tiles = call(packed, N, K, codes, both, 8, exact)
        launched.append(dev.last_dispatch())
    finally:
        dev.set_dispatch()
    assert np.array_equal(y.view(np.uint16), tiles.view(np.uint16))
    assert np.array_equal(again.view(np.uint16), tiles.view(np.uint16))
    assert launched == [want, want, (8, want[1])]
    assert int(exact[:16384].view(torch.int32).abs().sum()) == 0


@pytest.mark.parametrize("both", [False, True])
def test_equal_tokens_give_equal_rows(both):
    """A round of whole tiles and a tail behind it: the second half of the tokens is the first again."""
    M, K, N = 2048, 5120, 5120
    say(f"group order, equal tokens, both={both}")
    x16 = np.tile(synth.activations(M // 2, K, seed=7, outlier_frac=0.02), (2, 1))
    _, _, packed, codes = operands(M, K, N, both, x16=x16)
    y = call(packed, N, K, codes, both, 8, fq.make_workspace(M, N, K)).view(np.uint16)
    assert np.array_equal(y[:M // 2], y[M // 2:])


# (M, K, N, pieces): stage counts around the unrolled loop, tile edges; as in the 128-row form
@pytest.mark.parametrize("spin", [0, -1])
@pytest.mark.parametrize("both,bits", [(False, 6), (True, 8)])
@pytest.mark.parametrize("M,K,N,pieces", [
    (1, 128, 32, 1), (33, 256, 288, 2), (64, 384, 256, 3), (65, 512, 544, 1), (300, 640, 288, 5), (40, 768, 96, 6),
    (129, 896, 320, 7), (131, 1024, 256, 4), (96, 1408, 640, 11), (200, 2048, 32, 16)])
def test_half_height_tiles(M, K, N, pieces, both, bits, spin):
    say(f"64x256 group tiles M={M} K={K} N={N} pieces={pieces} both={both} A{bits} spin={spin}")
    w, x16, packed, codes = operands(M, K, N, both, bits)
    ws = fq.make_workspace(M, N, K, extra=((M + 63) // 64) * ((N + 255) // 256) * pieces << 16)
    dev.set_dispatch(2, pieces, 0, 19)
    dev.set_spin(spin)
    try:
        out = [call(packed, N, K, codes, both, bits, ws) for _ in range(2)]    # the counters are left zero
        assert dev.last_dispatch() == (19, pieces)
        assert int(ws[:16384].view(torch.int32).abs().sum()) == 0
    finally:
        dev.set_dispatch()
        dev.set_spin(0)
    assert np.array_equal(out[0].view(np.uint16), out[1].view(np.uint16))
    if both:
        _, _, ry, slack = reference(x16, w, bits)
        assert_close(out[0], ry, slack, "half height:")
    else:
        ref = oracle.linear(x16, w, bits, 128)
        assert_y_close(out[0], ref["y"], group_slack(ref))


# tile order because the codes do not fit LDS, or would crowd it; one or several rounds of workgroups
@pytest.mark.parametrize("bits", [6, 8])
@pytest.mark.parametrize("K,N", [(4096, 12288), (5120, 15360), (4096, 22016), (7680, 4096), (2048, 20512)])
def test_decode_from_fp16_and_from_codes(K, N, bits):
    say(f"group order, decode: K={K} N={N} A{bits}")
    w = synth.weights(N, K, 0.02, seed=K + N)
    packed = fq.pack_w6(*fq.quant_w6(to_dev(w), 128), 128)
    fn = fq.gemv_w6a6 if bits == 6 else fq.gemv_w6a8
    for M in (1, 2, 6, 11, 13, 16, 17, 24, 32):
        say(f"    {M} tokens")
        x = to_dev(synth.activations(M, K, seed=M, outlier_frac=0.02))
        xq, sx = fq.quant_act(x, bits)
        a = fn(packed, N, K, 128, x_fp16=x).cpu().numpy()
        b = fn(packed, N, K, 128, xq=xq, sx=sx).cpu().numpy()
        assert np.array_equal(a.view(np.uint16), b.view(np.uint16)), M


def check_scales_that_are_not_finite(cfg, both):
    """A packed weight scale may be infinite or NaN: a group whose sum is not zero gives that
    sign's infinity, a zero sum NaN, and no other channel notices."""
    M, K, N = 130, 640, 288
    say(f"group scales not finite: form {cfg}, both={both}")
    wq, sw = oracle.quantize(synth.weights(N, K, 0.02, seed=3), 6, 128)
    sw[3, 1] = sw[200] = np.inf
    sw[17, 0], sw[17, 4] = np.inf, -np.inf
    sw[50, 2] = np.nan
    x16 = synth.activations(M, K, seed=4, outlier_frac=0.02)
    x16[5] = 0.0
    x16[6, 128:256] = 0.0
    packed = fq.pack_w6(to_dev(wq), to_dev(sw), 128)
    xq, sx = oracle.quantize(x16.astype(np.float32), 8, 128 if both else 0)
    acc_g = oracle.matmul(xq, wq, 128)
    want = oracle.dequant_xgroup(acc_g, sx if both else np.repeat(sx.reshape(M, 1), K // 128, 1), sw).astype(np.float64)
    codes = (fq.quant_act_g128 if both else fq.quant_act)(to_dev(x16), 8)
    dev.set_dispatch(2, 1, 0, cfg)
    try:
        got = call(packed, N, K, codes, both, 8, fq.make_workspace(M, N, K, extra=8 << 20)).astype(np.float64)
        assert dev.last_dispatch()[0] == cfg
    finally:
        dev.set_dispatch()
    assert np.isposinf(want).any() and np.isneginf(want).any() and np.isnan(want).sum() >= M
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    fine = np.isfinite(want)
    assert np.allclose(got[fine], want[fine], rtol=2e-3, atol=2e-3)


@pytest.mark.parametrize("both", [False, True])
@pytest.mark.parametrize("cfg", [8, 18, 19])
def test_scales_that_are_not_finite(cfg, both):
    check_scales_that_are_not_finite(cfg, both)


# exactly a round of 128-row tiles; more: several items per workgroup, then the 14 (8) behind the round,
# whole or cut, 128 rows high (18) or 64 (19), at one to five stages and unequal pieces
@pytest.mark.parametrize("both,spin", [(False, 0), (False, -1), (True, 0), (True, -1)])
@pytest.mark.parametrize("M,K,N,cfg,pieces", [
    (1024, 256, 8192, 18, 1), (1029, 128, 7680, 18, 1), (1029, 256, 7680, 18, 2), (1029, 640, 7456, 18, 3), (33 * 128, 384, 1824, 18, 3),
    (1029, 128, 7680, 19, 1), (1029, 256, 7456, 19, 1), (1029, 640, 7456, 19, 4), (33 * 128, 384, 1824, 19, 2)])
def test_rounds_then_a_tail(M, K, N, cfg, pieces, both, spin):
    say(f"group tiles, a round and a tail: form {cfg} M={M} K={K} N={N} pieces={pieces} both={both} spin={spin}")
    w, x16, packed, codes = operands(M, K, N, both)
    ws = fq.make_workspace(M, N, K, extra=8 << 20)
    dev.set_dispatch(2, pieces, 0, cfg)
    dev.set_spin(spin)
    try:
        out = [call(packed, N, K, codes, both, 8, ws) for _ in range(2)]
        assert dev.last_dispatch() == (cfg, pieces)
        assert int(ws[:16384].view(torch.int32).abs().sum()) == 0
    finally:
        dev.set_dispatch()
        dev.set_spin(0)
    assert np.array_equal(out[0].view(np.uint16), out[1].view(np.uint16))
    if both:
        _, _, ry, slack = reference(x16, w, 8)
        assert_close(out[0], ry, slack, "a round and a tail:")
    else:
        ref = oracle.linear(x16, w, 8, 128)
        assert_y_close(out[0], ref["y"], group_slack(ref))


@pytest.mark.parametrize("cfg", [18, 19])
@pytest.mark.parametrize("both", [False, True])
def test_soak_of_the_fp32_hand_off(cfg, both):
    """1000 back-to-back calls on one workspace, every result compared bit for bit with the first,
    stopping at the first mismatch; the counters end at zero."""
    M, K, N, pieces = 100, 2304, 1120, 3
    say(f"soak: group tiles, form {cfg}, both={both}")
    _, _, packed, codes = operands(M, K, N, both)
    ws = fq.make_workspace(M, N, K, extra=8 << 20)

    def enqueue(out=None):
        if both:
            return dev.linear_g128(packed, N, K, *codes, workspace=ws, out=out)
        return dev.gemm_w6a8(packed, N, K, 128, xq=codes[0], sx=codes[1], workspace=ws, out=out)

    dev.set_dispatch(2, pieces, 0, cfg)
    try:
        first, y = enqueue(), torch.empty((M, N), dtype=torch.float16, device="cuda")
        assert dev.last_dispatch() == (cfg, pieces)
        differs = torch.zeros(1, dtype=torch.int32, device="cuda")
        for rep in range(1000):
            enqueue(y)
            differs += (y != first).any()
            if rep % 100 == 99:
                assert int(differs.item()) == 0, ("a call among", rep - 99, "..", rep, "differs")
    finally:
        dev.set_dispatch()
    assert int(ws[:16384].view(torch.int32).abs().sum()) == 0


@pytest.mark.parametrize("both", [False, True])
def test_graph_replay_of_the_half_height_tiles(both):
    """The quantizer and the library's own choice, tiles cut along K and a round with a tail,
    captured in one graph: three replays with fresh inputs, eager work in between."""
    say(f"group tiles, graph capture / replay, both={both}")
    cases = []
    for M, K, N, want in ((200, 4480, 1056, (19, 2)), (1029, 256, 7456, (19, 1))):
        w, _, packed, _ = operands(M, K, N, both)
        x = to_dev(synth.activations(M, K, seed=M))
        cases.append((M, K, N, want, w, packed, x, fq.make_workspace(M, N, K),
                      torch.empty((M, N), dtype=torch.float16, device="cuda")))

    def enqueue():
        for M, K, N, want, w, packed, x, ws, y in cases:
            if both:
                dev.linear_g128(packed, N, K, *fq.quant_act_g128(x, 8), workspace=ws, out=y)
            else:
                dev.gemm_w6a8(packed, N, K, 128, x_fp16=x, workspace=ws, out=y)
            assert dev.last_dispatch() == want

    enqueue()
    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            enqueue()
    torch.cuda.synchronize()
    for rep in range(3):
        for M, K, *_, x, ws, y in cases:
            x.copy_(to_dev(synth.activations(M, K, seed=100 * rep + M)))
        graph.replay()
        torch.cuda.synchronize()
        got = [c[-1].clone() for c in cases]
        enqueue()
        torch.cuda.synchronize()
        for c, g in zip(cases, got):
            assert torch.equal(c[-1], g), rep
    for c in cases:
        assert int(c[-2][:16384].view(torch.int32).abs().sum()) == 0
