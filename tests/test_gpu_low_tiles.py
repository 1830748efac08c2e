"""GPU parity of 128x256 tiles above 128 tokens: a whole round of 256 of them followed by tiles
cut along K in the same launch, and the sizes at which the library itself takes them."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_04405_amd as fq
from paper_2508_04405_amd import dev, synth

from gpu_helpers import assert_y_close, prepare, say, to_dev

pytestmark = pytest.mark.gpu


def check(M, K, N, dispatch, want, spin=0, stale=None):
    w = synth.weights(N, K, 0.02, seed=K)
    x = synth.activations(M, K, seed=M, outlier_frac=0.02)
    packed, _, _ = prepare(w)
    ref = oracle.linear(x, w, 6)
    ws = fq.make_workspace(M, N, K, extra=64 << 20)
    dev.set_dispatch(*dispatch)
    dev.set_spin(spin)
    try:
        for _ in range(2):
            if stale is not None:
                ws[16384:].fill_(stale)
            y, acc = dev.gemm_w6a6(packed, N, K, x_fp16=to_dev(x), workspace=ws, want_acc=True)
            assert dev.last_dispatch() == want
            assert np.array_equal(acc.cpu().numpy().astype(np.int64), ref["acc"])
            assert_y_close(y.cpu().numpy(), ref["y"])
        assert int(ws[:16384].view(torch.int32).abs().sum()) == 0
    finally:
        dev.set_dispatch()
        dev.set_spin(0)


# 256 tiles whole, then the remaining 14 (270 in all) or 1 cut in two or more
@pytest.mark.parametrize("spin", [0, -1])
@pytest.mark.parametrize("M,K,N,pieces,tail", [(1029, 256, 7680, 2, 14), (1029, 640, 7456, 5, 14), (33 * 128, 384, 1824, 3, 8)])
def test_round_then_cut(M, K, N, pieces, tail, spin):
    say(f"low tiles, a round then {tail} cut into {pieces}: M={M} K={K} N={N} spin={spin}")
    check(M, K, N, (2, pieces, 0, 16), (16, tail * pieces), spin)


# 256 items, one for every workgroup, and 288: 256-row tiles, low ones, 192-row ones
@pytest.mark.parametrize("cfg,M", [(12, 2048), (12, 2049), (15, 1024), (15, 1025), (20, 1536), (20, 1537)])
def test_one_round_and_more(cfg, M):
    say(f"one round of tiles and more: form {cfg} M={M}")
    check(M, 128, 8192, (2, 0, 0, cfg), (cfg, 1 if cfg == 12 else 0))


# One and several rows of low tiles and of 256-row tiles, one to all of the last row's slabs padding: what the
# area for the partial sums held before, sums of a larger call say, is nowhere added.
@pytest.mark.parametrize("spin", [0, -1])
@pytest.mark.parametrize("cfg,M,K,N,pieces", [
    (16, 1, 256, 288, 2), (16, 66, 640, 544, 5), (16, 96, 384, 256, 3), (16, 129, 512, 544, 4), (16, 161, 896, 288, 7),
    (16, 225, 1408, 256, 11), (16, 300, 2048, 32, 16), (13, 129, 640, 288, 5), (13, 300, 384, 544, 3)])
def test_padding_slabs(cfg, M, K, N, pieces, spin):
    say(f"padding slabs: form {cfg} M={M} K={K} N={N} pieces={pieces} spin={spin}")
    rows = 128 if cfg == 16 else 256
    wgs = (M + rows - 1) // rows * ((N + 255) // 256) * pieces
    check(M, K, N, (2, pieces, 0, cfg), (cfg, wgs), spin, stale=0x5b)


@pytest.mark.parametrize("M,K,N,want", [(129, 2048, 2048, 16), (300, 4096, 1056, 16), (600, 4096, 12288, 15), (100, 512, 40960, 15)])
def test_own_choice(M, K, N, want):
    say(f"low tiles by choice: M={M} K={K} N={N}")
    dev.gemm_w6a6(torch.zeros(fq.packed_bytes(N, K), dtype=torch.uint8, device="cuda"), N, K,
                  x_fp16=torch.zeros((M, K), dtype=torch.float16, device="cuda"))
    launched = dev.last_dispatch()
    assert launched[0] == want, launched
    check(M, K, N, (), launched)
