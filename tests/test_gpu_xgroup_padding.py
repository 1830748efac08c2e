"""Group-wise activation scales: the padded form's columns from M on are zero, the plain form leaves them."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2508_04405_amd as fq
from paper_2508_04405_amd import synth

from gpu_helpers import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [6, 8])
@pytest.mark.parametrize("M,K,stride", [(1, 128, 1), (1, 256, 64), (15, 128, 16), (16, 384, 17), (17, 640, 64),
                                        (64, 256, 64), (65, 1408, 130), (700, 1280, 704)])
def test_padding(M, K, stride, bits):
    say(f"group-wise scales, padding: M={M} K={K} stride={stride} A{bits}")
    x16 = synth.activations(M, K, seed=M + K, outlier_frac=0.02)
    x16[M // 2, :128] = 0.0
    want_q, want_s = oracle.quantize(x16.astype(np.float32), bits, 128)
    lib, x = fq.load(), to_dev(x16)
    for fn, beyond in ((lib.flexq_quant_act_g128_padded, 0.0), (lib.flexq_quant_act_g128, 7.0)):
        xq = torch.full((M, K), 99, dtype=torch.int8, device="cuda")
        sxg = torch.full((K // 128, stride), 7.0, dtype=torch.float16, device="cuda")
        assert fn(ctypes.c_void_p(x.data_ptr()), M, K, bits, xq.data_ptr(), sxg.data_ptr(), stride, None) == 0
        torch.cuda.synchronize()
        assert np.array_equal(xq.cpu().numpy(), want_q)
        got = sxg.cpu().numpy()
        assert np.array_equal(got[:, :M].view(np.uint16), want_s.T.view(np.uint16))
        assert np.all(got[:, M:] == beyond)
