"""GPU parity of the weight quantizer and packer at the row lengths where the quantizer changes
its workgroup, with ragged last chunks, and on pointers aligned to one element only."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2508_04405_amd as fq
from paper_2508_04405_amd import synth

from gpu_helpers import say, to_dev

pytestmark = pytest.mark.gpu


def ragged_weights(N, K, seed):
    w = synth.weights(N, K, 0.02, seed=seed)
    w[1] = 0.0                                            # an all-zero row
    w[2, -1] = 5.0                                        # the absmax in the last chunk
    w[3] = ((np.arange(K) % 62 - 31) + 0.5) * 0.25        # ties
    w[3, 0] = 31 * 0.25
    w[4] *= 1e-6                                          # the fp16 scale is subnormal
    w[5] *= 1e9                                           # the fp16 scale is infinite: codes 0
    w[6] *= 1e-30                                         # it underflows: scale 1, codes 0
    return w


@pytest.mark.parametrize("group", [0, 128])
@pytest.mark.parametrize("K", [128, 2048, 2176, 4224, 8320, 16512, 32896, 65536])
def test_quant_and_pack_rows(K, group):
    say(f"quant_w6 + pack_w6 K={K} group={group}")
    N = 32
    w = ragged_weights(N, K, seed=K)
    rq, rs = oracle.quantize(w, 6, group)
    loose = torch.empty(N * K + 1, dtype=torch.float32, device="cuda")[1:]        # 4-byte aligned only
    loose.copy_(to_dev(w).view(-1))
    for src in (to_dev(w), loose.view(N, K)):
        wq, sw = fq.quant_w6(src, group)
        assert np.array_equal(wq.cpu().numpy(), rq)
        assert np.array_equal(sw.cpu().numpy().view(np.uint16), rs.view(np.uint16))
    back, back_s = fq.unpack_w6(fq.pack_w6(wq, sw, group), N, K, group)
    assert np.array_equal(back.cpu().numpy(), rq)
    assert np.array_equal(back_s.cpu().numpy().view(np.uint16), rs.view(np.uint16))


def test_quant_codes_at_an_odd_address():
    say("quant_w6 into codes at an odd address")
    N, K = 32, 640
    w = ragged_weights(N, K, seed=1)
    rq, _ = oracle.quantize(w, 6, 0)
    buf = torch.zeros(N * K + 2, dtype=torch.int8, device="cuda")
    sw = torch.empty(N, dtype=torch.float16, device="cuda")
    vp = ctypes.c_void_p
    assert fq.load().flexq_quant_w6(vp(to_dev(w).data_ptr()), N, K, 0, vp(buf.data_ptr() + 1), vp(sw.data_ptr()),
                                    vp(torch.cuda.current_stream().cuda_stream)) == 0
    got = buf.cpu().numpy()
    assert np.array_equal(got[1:-1].reshape(N, K), rq) and got[0] == 0 and got[-1] == 0
