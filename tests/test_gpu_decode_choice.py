"""GPU parity of the library's own choice for batched decode at the sizes where it changes: K
splits that fill whole rounds of 256 workgroups, activations quantized into tile order although
they would fit LDS, four wavefronts per workgroup."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_04405_amd import dev, synth

from gpu_helpers import assert_y_close, group_slack, prepare, say, to_dev

pytestmark = pytest.mark.gpu


# want: (1, K splits, 500 more with the activations in tile order)
@pytest.mark.parametrize("M,K,N,bits,want", [
    (11, 7680, 4096, 8, 1), (12, 7680, 4096, 8, 2), (16, 7680, 4096, 6, 502), (20, 7680, 4096, 6, 502),
    (32, 7680, 4096, 8, 502), (15, 11520, 5120, 6, 1), (16, 11520, 5120, 6, 503), (32, 11520, 5120, 8, 503),
    (12, 4096, 4096, 6, 1), (13, 4096, 4096, 6, 501), (16, 4096, 4096, 8, 501), (12, 2048, 20512, 8, 1), (32, 15360, 10240, 8, 503),
    (32, 2048, 20512, 6, 501)])
def test_own_choice(M, K, N, bits, want):
    say(f"own choice: M={M} K={K} N={N} A{bits}")
    w = synth.weights(N, K, 0.02, seed=K)
    x = synth.activations(M, K, seed=M, outlier_frac=0.02)
    packed, _, _ = prepare(w)
    ref = oracle.linear(x, w, bits)
    fn = dev.gemv_w6a6 if bits == 6 else dev.gemv_w6a8
    y, acc = fn(packed, N, K, x_fp16=to_dev(x), want_acc=True)
    assert dev.last_dispatch() == (1, want)
    assert np.array_equal(acc.cpu().numpy().astype(np.int64), ref["acc"])
    assert_y_close(y.cpu().numpy(), ref["y"])


@pytest.mark.parametrize("M,bits", [(16, 6), (24, 8)])
def test_group_scales_with_splits(M, bits):
    say(f"own choice, group scales: M={M} A{bits}")
    K, N = 7680, 4096
    w = synth.weights(N, K, 0.02, seed=3)
    x = synth.activations(M, K, seed=M, outlier_frac=0.02)
    packed, _, _ = prepare(w, 128)
    ref = oracle.linear(x, w, bits, 128)
    fn = dev.gemv_w6a6 if bits == 6 else dev.gemv_w6a8
    y = fn(packed, N, K, 128, x_fp16=to_dev(x))
    torch.cuda.synchronize()
    assert dev.last_dispatch()[1] % 500 == 2
    assert_y_close(y.cpu().numpy(), ref["y"], group_slack(ref))
