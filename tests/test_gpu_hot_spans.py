"""The hot IDs' pass at the sizes that choose hot IDs by themselves: runs that
fill their chunks exactly, by one occurrence less and by one more, at the sizes
and widths where the occurrences per lane group change (32 to 128).  The runs
are long enough for the sort's sample to find their IDs, which is checked."""
import pytest
import torch

import paper_2205_11048_amd as gba

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _sampled(ids, n, first_only):
    """IDs at the positions the sort samples: 256 runs of 64 spread over the
    input; an ID is found among the first 64 runs and then counted in all."""
    run = torch.arange(64 if first_only else 256, device=DEV)
    p0 = ((2 * run + 1) * n // 512 - 32).clamp_(0, n - 64)
    return ids[(p0[:, None] + torch.arange(64, device=DEV)).flatten()]


@pytest.mark.parametrize("N,D,span", [((1 << 22) + 5, 32, 32), ((1 << 22) + 5, 16, 32), (5_000_011, 64, 64),
                                      ((1 << 22) + 5, 100, 128), ((1 << 22) + 5, 256, 128), ((1 << 24) - 1, 32, 32),
                                      ((1 << 24) + 3, 32, 64), ((1 << 24) + 3, 64, 128), ((1 << 25) - 1, 4, 32),
                                      ((1 << 25) + 3, 4, 128)])
def test_hot_runs_that_end_at_chunks(N, D, span):
    K, R = 6, 3_000_000 if D < 64 else 300_000
    lanes = 1
    while lanes * 4 < D:
        lanes *= 2
    chunk = 4 * (64 // lanes) * span                       # occurrences per block of the pass
    long = 16 * chunk
    while long < N // 256:                                 # some 64 of the 16,384 sampled positions
        long *= 2
    g = torch.Generator(device=DEV).manual_seed(N)
    ids = torch.randint(0, R, (N,), device=DEV, generator=g)
    at = torch.randperm(N, device=DEV, generator=g)
    start = 0
    planted = ((11, long), (R // 2, long - 1), (R - 1, long + 1), (77_777, max(40_000, N // 512)))
    for hot, n in planted:
        ids[ids == hot] = hot + 1 if hot + 1 < R else 12
        ids[at[start:start + n]] = hot
        start += n
    for hot, _ in planted:
        assert int((_sampled(ids, N, True) == hot).sum()) >= 1 and int((_sampled(ids, N, False) == hot).sum()) >= 8
    cut = torch.randint(0, N + 1, (K - 1,), device=DEV, generator=g).sort().values
    zero = torch.zeros(1, dtype=torch.int64, device=DEV)
    off = torch.cat([zero, cut, zero + N])
    rows = torch.randint(-64, 65, (N, D), device=DEV, generator=g).to(torch.float32) / 64   # exact sums
    tokens = torch.tensor([9, 5, 9, 8, 9, 9], device=DEV)
    w = torch.tensor([1.0, 0.0, 0.5, 1.0, 1.0, 1.0], device=DEV)
    out = [torch.full((N,), -5, dtype=torch.int64, device=DEV), torch.full((N + 1,), -5, dtype=torch.int64, device=DEV),
           torch.full((N,), -5, dtype=torch.int32, device=DEV), torch.full((N,), -5, dtype=torch.int32, device=DEV),
           torch.empty((N, D), device=DEV), torch.zeros(1, dtype=torch.int64, device=DEV)]
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = torch.empty(gba.gba_aggregate_sparse_workspace_size(N, K, D, R), dtype=torch.uint8, device=DEV)
    gba.gba_aggregate_sparse(ids, rows, off, R, w, tokens, 9, 3, None, gba.DECAY_TOKEN, gba.NORM_BY_K, *out, ws, err)
    unique, inverse, count = torch.unique(ids, return_inverse=True, return_counts=True)
    U = unique.numel()
    m = torch.searchsorted(off[1:].contiguous(), torch.arange(N, device=DEV), right=True)
    pairs = torch.unique(inverse * K + m)
    live = pairs[w[pairs % K] != 0]
    sums = torch.zeros((U, D), dtype=torch.float64, device=DEV)
    for a in range(0, N, 1 << 21):
        b = min(N, a + (1 << 21))
        sums.index_add_(0, inverse[a:b], rows[a:b].double() * w[m[a:b], None])
    assert int(err.item()) == 0 and int(out[5].item()) == U
    assert torch.equal(out[0][:U], unique)
    assert torch.equal(out[1][:U + 1], torch.cat([zero, count.cumsum(0)]))
    assert torch.equal(out[2][:U].to(torch.int64), torch.bincount(pairs // K, minlength=U))
    assert torch.equal(out[3][:U].to(torch.int64), torch.bincount(live // K, minlength=U))
    assert torch.equal(out[4][:U], (sums / K).float())
