"""Group-128 scales above 128 tokens on layers of few tiles: K is cut where the weights' bytes alone
would leave it whole.  The library's choice at the sizes where it changes, against the 128x128
tiles with the same K splits (the same bits, whatever the workspace) and the CPU oracle."""
import numpy as np
import pytest

import oracle
import paper_2508_04405_amd as fq
from paper_2508_04405_amd import dev

from gpu_helpers import assert_y_close, group_slack, say
from test_gpu_group_order import call, operands
from test_gpu_xgroup import assert_close, reference

pytestmark = pytest.mark.gpu


# want: form and K splits -- half height, 128 rows high because half height no longer fits a round, cut
# anew though cut before; rows and columns that end inside a tile; stages that do not divide
@pytest.mark.parametrize("both", [False, True])
@pytest.mark.parametrize("M,K,N,want", [
    (1000, 3328, 32, (19, 4)), (300, 4096, 1088, (19, 4)), (1101, 4096, 512, (19, 4)), (500, 8576, 96, (19, 7)),
    (1029, 4224, 2592, (19, 1)), (700, 13824, 5120, (18, 2))])
def test_few_tiles_are_cut(M, K, N, want, both):
    say(f"group split: M={M} K={K} N={N} both={both}")
    w, x16, packed, codes = operands(M, K, N, both)
    exact, roomy = fq.make_workspace(M, N, K), fq.make_workspace(M, N, K, extra=64 << 20)
    y = call(packed, N, K, codes, both, 8, exact)
    assert dev.last_dispatch() == want
    assert np.array_equal(call(packed, N, K, codes, both, 8, roomy).view(np.uint16), y.view(np.uint16))
    dev.set_dispatch(2, 0, 0, 8)
    try:
        tiles = call(packed, N, K, codes, both, 8, exact)
        assert dev.last_dispatch() == (8, want[1])
    finally:
        dev.set_dispatch()
    assert np.array_equal(tiles.view(np.uint16), y.view(np.uint16))
    if M * K * N > 2e10:       # (the forms agree; the oracle would take a minute)
        return
    if both:
        _, _, ry, slack = reference(x16, w, 8)
        assert_close(y, ry, slack, "cut:")
    else:
        ref = oracle.linear(x16, w, 8, 128)
        assert_y_close(y, ref["y"], group_slack(ref))
