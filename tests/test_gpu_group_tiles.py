"""GPU parity of the persistent tiles for group-128 scales (forced through the development
library) against the CPU oracle: one to several stages, tiles whole and cut along K, ragged
tokens and columns, per-token and per-group activation scales."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_04405_amd as fq
from paper_2508_04405_amd import dev, synth

from gpu_helpers import assert_y_close, group_slack, say, to_dev
from test_gpu_xgroup import assert_close, reference

pytestmark = pytest.mark.gpu

# (M, K, N, pieces): stage counts around the unrolled loop (1 .. 8, 11), tile edges, one row
# block and one row beyond it, columns that end inside a tile, every number of pieces once
CASES = [(1, 128, 32, 1), (33, 256, 288, 2), (128, 384, 256, 3), (129, 512, 544, 1), (300, 640, 288, 5),
         (40, 768, 96, 6), (257, 896, 320, 7), (131, 1024, 256, 4), (96, 1408, 640, 11), (200, 2048, 32, 16)]


def run(M, K, N, pieces, both, bits, spin=0):
    w = synth.weights(N, K, 0.02, seed=K + N)
    x16 = synth.activations(M, K, seed=M, outlier_frac=0.02)
    packed = fq.pack_w6(*fq.quant_w6(to_dev(w), 128), 128)
    ws = fq.make_workspace(M, N, K, extra=((M + 127) // 128) * ((N + 255) // 256) * pieces << 17)
    dev.set_dispatch(2, pieces, 0, 18)
    dev.set_spin(spin)
    try:
        out = []
        for _ in range(2):                     # twice on one workspace: its counters are left zero
            if both:
                xq, sx = fq.quant_act_g128(to_dev(x16), bits)
                out.append(dev.linear_g128(packed, N, K, xq, sx, workspace=ws).cpu().numpy())
            else:
                fn = dev.gemm_w6a6 if bits == 6 else dev.gemm_w6a8
                out.append(fn(packed, N, K, 128, x_fp16=to_dev(x16), workspace=ws).cpu().numpy())
            assert dev.last_dispatch() == (18, pieces)
        assert int(ws[:16384].view(torch.int32).abs().sum()) == 0
    finally:
        dev.set_dispatch()
        dev.set_spin(0)
    # the partial sums are added in the order of the pieces whoever adds them
    assert np.array_equal(out[0].view(np.uint16), out[1].view(np.uint16))
    return w, x16, out[0]


@pytest.mark.parametrize("both,bits", [(False, 6), (False, 8), (True, 6), (True, 8)])
@pytest.mark.parametrize("M,K,N,pieces", CASES)
def test_group_tiles(M, K, N, pieces, both, bits):
    say(f"group tiles M={M} K={K} N={N} pieces={pieces} both={both} A{bits}")
    w, x16, y = run(M, K, N, pieces, both, bits)
    if both:
        _, _, ry, slack = reference(x16, w, bits)
        assert_close(y, ry, slack, "group tiles:")
    else:
        ref = oracle.linear(x16, w, bits, 128)
        assert_y_close(y, ref["y"], group_slack(ref))


@pytest.mark.parametrize("spin", [-1, 1])
@pytest.mark.parametrize("both", [False, True])
def test_group_tiles_pieces_that_do_not_wait(both, spin):
    """Pieces that give up waiting leave their slabs to others: the same bits."""
    say(f"group tiles, spin {spin}, both={both}")
    want = run(300, 1280, 544, 5, both, 8)[2]
    got = run(300, 1280, 544, 5, both, 8, spin)[2]
    assert np.array_equal(got.view(np.uint16), want.view(np.uint16))
