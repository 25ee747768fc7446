"""The hot IDs' pass at the sizes that choose hot IDs by themselves: runs that
fill their chunks exactly, by one occurrence less and by one more, at both
ends of the size from which a lane group takes 128 occurrences instead of 32."""
import pytest
import torch

import paper_2205_11048_amd as gba

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("N,D", [((1 << 22) + 5, 32), ((1 << 22) + 5, 16), (5_000_011, 64), ((1 << 25) - 1, 4),
                                 ((1 << 25) + 3, 4)])
def test_hot_runs_that_end_at_chunks(N, D):
    K, R = 6, 3_000_000
    span = 128 if N >= 1 << 25 else 32
    lanes = 1
    while lanes * 4 < D:
        lanes *= 2
    chunk = 4 * (64 // lanes) * span                       # occurrences per block of the pass
    g = torch.Generator(device=DEV).manual_seed(N)
    ids = torch.randint(0, R, (N,), device=DEV, generator=g)
    at = torch.randperm(N, device=DEV, generator=g)
    start = 0
    for hot, n in ((11, 4 * chunk), (1_500_000, 4 * chunk - 1), (R - 1, 4 * chunk + 1), (77_777, 40_000)):
        ids[ids == hot] = hot + 1 if hot + 1 < R else 12
        ids[at[start:start + n]] = hot
        start += n
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
