"""The 192 x 256 tiles of the GEMM with both operands through LDS, against the CPU oracle: int32 sums
bit-exact, fp16 outputs within one fp16 ulp."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_04405_amd as fq
from paper_2508_04405_amd import dev, synth

from gpu_helpers import DEV, assert_y_close, prepare, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(1, 128, 32),            # one stage, one row, an eighth of the columns
                                   (191, 256, 256), (192, 384, 288), (193, 512, 224),    # the tile's edges
                                   (97, 640, 544),          # the second wavefront row holds one token
                                   (577, 1280, 1120),       # four rows of tiles, the last with one token
                                   (385, 384, 25600)])      # 300 tiles: two per workgroup for some
@pytest.mark.parametrize("bits", [6, 8])
def test_against_the_oracle(M, K, N, bits):
    say(f"192x256 tiles M={M} K={K} N={N} bits={bits}")
    w = synth.weights(N, K, 0.02, seed=91)
    x = synth.activations(M, K, seed=92, outlier_frac=0.02)
    packed, _, _ = prepare(w)
    xq, sx = fq.quant_act(to_dev(x), bits)
    ref = oracle.linear(x, w, bits)
    call = dev.gemm_w6a6 if bits == 6 else dev.gemm_w6a8
    out = torch.full((M + 192, N), float("nan"), dtype=torch.float16, device=DEV)
    dev.set_dispatch(2, 1, 0, 20)
    try:
        y, acc = call(packed, N, K, xq=xq, sx=sx, want_acc=True)
        assert dev.last_dispatch()[0] == 20
        call(packed, N, K, xq=xq, sx=sx, out=out[:M])
        torch.cuda.synchronize()
    finally:
        dev.set_dispatch(0, 0, 0, 0)
    assert np.array_equal(acc.cpu().numpy().astype(np.int64), ref["acc"])
    assert_y_close(y.cpu().numpy().view(np.float16), ref["y"])
    assert_y_close(out[:M].cpu().numpy().view(np.float16), ref["y"])
    assert bool(torch.isnan(out[M:]).all())                 # nothing is stored beyond the last token


def test_where_the_dispatch_takes_them():
    """Tokens that 256-row tiles would pad by half, and neighbours that stay with those."""
    say("192x256 tiles by dispatch")
    for M, N, K, taken in ((576, 15360, 5120, True), (1152, 8192, 8192, True), (512, 15360, 5120, False),
                           (1024, 8192, 8192, False)):
        packed = torch.zeros(fq.packed_bytes(N, K, 0), dtype=torch.uint8, device=DEV)
        xq = torch.zeros((M, K), dtype=torch.int8, device=DEV)
        dev.gemm_w6a8(packed, N, K, 0, xq=xq, sx=torch.ones((M,), dtype=torch.float16, device=DEV))
        torch.cuda.synchronize()
        assert (dev.last_dispatch()[0] == 20) == taken, (M, N, K, dev.last_dispatch())
