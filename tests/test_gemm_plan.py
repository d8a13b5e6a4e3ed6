"""Scratch of the projections' K split (host only): the split does not change
within a block of rows, so a buffer sized for a block's last row holds every
shorter call, as the workspace assumes."""
import pytest

import paper_2410_20290_amd as sr


@pytest.mark.parametrize("N,K,mode", [(6144, 4096, 0), (4096, 14336, 1), (14336, 4096, 2), (2048, 8192, 1),
                                      (1536, 512, 2), (512, 1536, 0), (8192, 512, 0), (384, 320, 0)])
def test_split_is_constant_within_a_block_of_rows(N, K, mode):
    scratch = lambda M: int(sr.lib().sr_projection_scratch(sr.SR_BF16, M, N, K, mode))
    ends = [0, 32, 64, 112, 128] + list(range(256, 6401, 128))
    for lo, hi in zip(ends, ends[1:]):
        per_row = {scratch(M) / M for M in range(lo + 1, hi + 1)}
        assert len(per_row) == 1, (lo, hi, per_row)
