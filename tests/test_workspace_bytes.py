"""The workspace a batched decode call asks for: counters, the codes and scales of its own quantizer,
and partial sums for the splits of the tiled kernel, which the streaming kernel's splits share.  The
splits that fill whole rounds of workgroups must not make it larger."""
import pytest

from paper_2508_04405_amd import binding


@pytest.mark.parametrize("M,N,K,splits", [
    (16, 10240, 15360, 3), (32, 10240, 15360, 3), (12, 4096, 11008, 8), (32, 4096, 11008, 8), (24, 2048, 16384, 16),
    (32, 5120, 13824, 6)])
def test_workspace_bytes(M, N, K, splits):
    assert binding.workspace_bytes(M, N, K) == 16384 + 32 * K + 256 + splits * M * N * 4
