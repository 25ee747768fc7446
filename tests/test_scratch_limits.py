"""Sizes that gba_aggregate_sparse_noalloc takes: the workspace of every size
up to these stays within the library's fixed scratch array (host query, no GPU)."""
import pytest

import paper_2205_11048_amd as gba

# width -> the largest number of occurrences whose workspace fits
LARGEST = {4: 2_708_608, 8: 2_704_896, 12: 2_695_936, 16: 2_691_839, 20: 2_667_008, 32: 2_643_904, 36: 2_568_704,
           64: 2_473_280, 68: 2_256_128, 128: 1_971_712, 132: 1_532_672, 256: 1_090_560}


@pytest.mark.parametrize("D", sorted(LARGEST))
@pytest.mark.parametrize("R", [1, 1000, 1 << 17, 1 << 20, 1 << 24, 1 << 27, 1 << 32])
def test_workspace_stays_within_the_fixed_array(D, R):
    most = LARGEST[D]
    sizes = {most - k for k in range(0, 2048, 63)}
    sizes |= {int(most * f) for f in (0.01, 0.1, 0.2, 0.3, 0.4, 0.5, 0.6, 0.7, 0.8, 0.9, 0.95, 0.99)}
    sizes |= {min(most, (1 << b) + d) for b in range(10, 22) for d in (-1, 0, 1)}
    for N in sorted(sizes):
        assert gba.gba_aggregate_sparse_workspace_size(N, 64, D, R) <= gba.NOALLOC_SCRATCH_BYTES, N
