"""Workspace queries (host only, no GPU): scratch sized for the largest input
serves every smaller one, at every size where a plan, a digit width, a tile or
a lane group's span changes, and whatever the table's size where the sort has
no hot-key plan; and the fixed array of the no-allocation call holds what it
held when the small sort's counts had room of their own."""
import random

import pytest

import paper_2205_11048_amd as gba


def _sizes():
    rng = random.Random(7)
    out = set(range(0, 40))
    for b in range(4, 28):
        out |= {(1 << b) + d for d in (-4097, -2049, -1025, -1024, -257, -65, -1, 0, 1, 64, 257, 1024, 2049, 4097)}
    out |= {(1 << 20) - 37_889, (1 << 20) - 19_713, 4095 * 1024, 4095 * 1024 + 1, 243_300, 29_500_000, 31_800_000}
    x = 50.0
    while x < (1 << 28) - 1:
        out.add(int(x))
        x *= 1.0 + 0.03 * rng.random()
    return sorted(n for n in out if 0 <= n < (1 << 28))


SIZES = _sizes()


def _assert_never_falls(query, what):
    most, at = 0, 0
    for n in SIZES:
        b = query(n)
        assert b >= most, f"{what}: {b} bytes for {n}, {most} for {at}"
        most, at = b, n


@pytest.mark.parametrize("R", [1, 200, 5_000, 1 << 17, 1 << 20, 10_000_000, 100_000_000, 1 << 32])
def test_sort_and_pull_queries_never_fall(R):
    _assert_never_falls(lambda n: gba.gba_pull_workspace_size(n, R), "pull")
    for plan in (gba.SORT_AUTO, gba.SORT_PLAIN, gba.SORT_HOT):
        _assert_never_falls(lambda n: gba.gba_sort_ids_workspace_size(n, R, plan), f"sort, plan {plan}")


@pytest.mark.parametrize("R", [1, 1 << 18, 10_000_000, 1 << 32])
@pytest.mark.parametrize("D", [4, 8, 12, 16, 32, 64, 100, 128, 256])
def test_sparse_queries_never_fall(D, R):
    for plan in (gba.SORT_AUTO, gba.SORT_PLAIN, gba.SORT_HOT):
        _assert_never_falls(lambda n: gba.gba_aggregate_sparse_plan_workspace_size(n, 50, D, R, plan),
                            f"sparse, plan {plan}")
    _assert_never_falls(lambda n: gba.gba_aggregate_apply_sparse_workspace_size(n, 50, D, R, "adam"), "fused")


@pytest.mark.parametrize("n", [1, 20_000, 33_000, 300_000, 700_000, 1_100_000, 1_900_000, 2_500_000, (1 << 22) - 1])
def test_plain_queries_do_not_depend_on_the_table(n):
    """Below the sizes that choose hot IDs one workspace serves tables of any size."""
    for query in (lambda R: gba.gba_pull_workspace_size(n, R),
                  lambda R: gba.gba_sort_ids_workspace_size(n, R, gba.SORT_AUTO),
                  lambda R: gba.gba_aggregate_sparse_workspace_size(n, 8, 32, R)):
        assert len({query(1 << b) for b in range(33)}) == 1


@pytest.mark.parametrize("D,N", [(144, 1_475_007), (188, 1_295_935)])
def test_fixed_array_at_the_largest_sizes(D, N):
    """Sizes that filled the array to its last kilobyte."""
    for b in range(33):
        assert gba.gba_aggregate_sparse_workspace_size(N, 64, D, 1 << b) <= gba.NOALLOC_SCRATCH_BYTES, b


@pytest.mark.gpu
@pytest.mark.parametrize("n", [5_000, 33_001, 300_007, (1 << 19) - 1, 1_023_500, (1 << 20) + 5, (1 << 21) + 1])
def test_calls_stay_inside_the_queried_bytes(n):
    """A workspace queried for n and one queried for more both serve n, and no
    byte past the queried ones is written (the small sort's counts end inside
    the scratch of the passes that follow)."""
    import torch
    R, D, K, pad = 1 << 20, 16, 3, 1 << 20
    g = torch.Generator(device="cuda").manual_seed(n)
    ids = (torch.rand(n, device="cuda", generator=g).pow(4) * R).to(torch.int64)
    rows = torch.randint(-64, 65, (n, D), device="cuda", generator=g).float() / 64
    off = torch.tensor([0, n // 3, n // 2, n], device="cuda")
    w = torch.tensor([1.0, 0.5, 1.0], device="cuda")
    tokens = torch.full((K,), 9, device="cuda")
    table = torch.arange(R * 4, device="cuda", dtype=torch.float32).reshape(R, 4)
    unique, inverse = torch.unique(ids, return_inverse=True)
    U = unique.numel()
    j = torch.arange(n, device="cuda")
    sums = torch.zeros((U, D), dtype=torch.float64, device="cuda")
    sums.index_add_(0, inverse, rows.double() * w[torch.searchsorted(off[1:], j, right=True), None])
    for size in (n, min(n + 40_000, 3 * n)):
        need = gba.gba_aggregate_sparse_workspace_size(size, K, D, R)
        ws = torch.full((need + pad,), 0xA5, dtype=torch.uint8, device="cuda")
        out = [torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(n + 1, dtype=torch.int64, device="cuda"),
               torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda"),
               torch.empty((n, D), device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")]
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        gba.gba_aggregate_sparse(ids, rows, off, R, w, tokens, 9, 3, None, gba.DECAY_TOKEN, gba.NORM_BY_K, *out,
                                 ws[:need], err)
        assert int(err.item()) == 0 and int(out[5].item()) == U
        assert torch.equal(out[0][:U], unique) and torch.equal(out[4][:U], (sums / K).float())
        assert bool((ws[need:] == 0xA5).all())
        need = gba.gba_pull_workspace_size(size, R)
        ws = torch.full((need + pad,), 0xA5, dtype=torch.uint8, device="cuda")
        got = torch.empty(n, dtype=torch.int32, device="cuda")
        got_rows = torch.empty((n, 4), device="cuda")
        gba.gba_pull_rows(ids, table, out[0], got, got_rows, out[5], ws[:need], err)
        assert int(err.item()) == 0 and int(out[5].item()) == U
        assert torch.equal(got.long(), inverse) and torch.equal(got_rows[:U], table[unique])
        assert bool((ws[need:] == 0xA5).all())
