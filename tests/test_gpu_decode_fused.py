"""fp16 activations quantized inside the streaming kernel by the library's own choice, around the sizes
where it stops doing so: codes and sums exact, the result that of a quantizer launch ahead."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_04405_amd as fq
from paper_2508_04405_amd import dev, synth

from gpu_helpers import prepare, say, to_dev

pytestmark = pytest.mark.gpu


# one to eight tokens; less than a wavefront's lanes of values, several loads a lane, one and two rounds of
# workgroups, K splits
@pytest.mark.parametrize("group", [0, 128])
@pytest.mark.parametrize("K,N", [(128, 32), (384, 96), (640, 8224), (1280, 288), (1408, 16384), (4096, 512), (5120, 96)])
def test_fused_equals_separate(K, N, group):
    w = synth.weights(N, K, 0.02, seed=K + N)
    packed, wq, _ = prepare(w, group)
    for bits in (6, 8):
        fn = dev.gemv_w6a6 if bits == 6 else dev.gemv_w6a8
        for M in (1, 2, 3, 4, 5, 7, 8):
            say(f"fused by choice: K={K} N={N} M={M} A{bits} group={group}")
            x16 = synth.activations(M, K, seed=M, outlier_frac=0.02)
            x16[M // 2] = 0.0
            x = to_dev(x16)
            out = []
            for fuse in (2, 0, 1):
                dev.set_fuse(fuse)
                try:
                    out.append(fn(packed, N, K, group, x_fp16=x))
                finally:
                    dev.set_fuse(0)
            assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2]), (M, bits)
            if group == 0:
                xq, _ = oracle.quantize(x16.astype(np.float32), bits)
                _, acc = fn(packed, N, K, group, x_fp16=x, want_acc=True)
                assert np.array_equal(acc.cpu().numpy(), oracle.matmul(xq, wq.cpu().numpy()))
