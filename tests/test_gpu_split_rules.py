"""The edges of the rules that split the work of the segment passes: the
positions per lane group of the row pass at small sizes, and the groups of
1024-position tiles in which run heads are numbered (groups of 4 tiles, of 16
from 4096 tiles, added up by every block to 1024 groups and scanned beyond)."""
import numpy as np
import pytest
import torch

import paper_2205_11048_amd as gba
from compare import assert_exact
from synth import counter
from synth import workload
from test_gpu_parity import _check_sparse, _run_sparse, _sparse_step, _table_and_state, dev
import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("D,N", [(4, 20_011), (4, 262_143), (4, 262_144), (16, 20_480), (16, 131_073),
                                 (32, 4_099), (32, 140_001), (64, 66_001), (256, 1_025), (256, 70_003)])
def test_row_spans_of_small_inputs(D, N):
    """Lane groups of 8, 16 and 32 positions (and the size from which 32 is
    always taken), with segments that end inside a group, at its end, in later
    groups and in later tiles; dyadic rows make every sum exact."""
    K, R = 5, 4_000
    rng = np.random.default_rng(N)
    ids = rng.integers(0, R, N)
    ids[rng.random(N) < 0.25] = 1234                       # a segment over many tiles
    ids[rng.random(N) < 0.1] = 77                          # and over many groups
    cut = np.sort(rng.integers(0, N + 1, K - 1))
    off = np.concatenate([[0], cut, [N]]).astype(np.int64)
    rows = counter.values_range(N, counter.STREAM_ROWS, 0, N * D, counter.KIND_DYADIC).reshape(N, D)
    tokens = 60 - np.array([0, 4, 1, 2, 0])
    w, _, _ = oracle.token_weights(tokens, 60, 2)
    res = _run_sparse(ids.astype(np.int64), rows, off, w, tokens, 60, 2, R)
    _check_sparse(res, ids, rows, off, w, tokens, 60, 2, expect_exact=True)


@pytest.mark.parametrize("n,D", [(n, 4) for n in (1, 1023, 1024, 1025, 4096, 4097, 16_385, (1 << 19) - 1, 1 << 19, 1_048_577,
                                                 4096 * 1024 - 1025, 4096 * 1024 + 1, 16 * 1024 * 1024 + 1,
                                                 17 * 1024 * 1024 + 1025, (1 << 25) + 1025)] +
                         [(257, 32), (3 * 1024 * 1024 - 1, 32), (3 * 1024 * 1024 + 1, 24), (600_001, 12),
                          (1 << 25, 8)])
def test_run_numbers_over_tile_groups(n, D):
    """Every position's run number, across tiles, groups of tiles, the sizes
    from which a block takes a whole tile, from which the group counts are
    scanned by a launch of their own and from which the rows are gathered by one."""
    R = 3_000_000
    g = torch.Generator(device=DEV).manual_seed(n)
    ids = torch.randint(0, R, (n,), device=DEV, generator=g)
    table = torch.arange(R * D, device=DEV, dtype=torch.float32).reshape(R, D)
    unique = torch.full((n,), -5, dtype=torch.int64, device=DEV)
    inverse = torch.full((n,), -5, dtype=torch.int32, device=DEV)
    rows = torch.empty((n, D), device=DEV)
    num = torch.full((1,), -5, dtype=torch.int64, device=DEV)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = torch.empty(gba.gba_pull_workspace_size(n, R), dtype=torch.uint8, device=DEV)
    gba.gba_pull_rows(ids, table, unique, inverse, rows, num, ws, err)
    ref, ref_inverse = torch.unique(ids, return_inverse=True)
    U = ref.numel()
    assert int(err.item()) == 0 and int(num.item()) == U
    assert torch.equal(unique[:U], ref)
    assert torch.equal(inverse.to(torch.int64), ref_inverse)
    assert torch.equal(rows[:U], table[ref])


@pytest.mark.parametrize("plan", [gba.SORT_PLAIN, gba.SORT_HOT])
@pytest.mark.parametrize("N", [1024, 4097, 1_048_575])
def test_segments_over_tile_groups(N, plan):
    """Segment numbers, starts and counts at the same edges, on both plans (with
    hot IDs below, between and above the cold ones)."""
    K, D, R = 3, 4, 50_000
    rng = np.random.default_rng(N)
    ids = rng.integers(5, R - 5, N)
    for k, hot in enumerate((0, 1, 25_000, R - 2, R - 1)):
        ids[rng.random(N) < 0.08] = hot
    off = np.array([0, N // 3, N // 2, N], np.int64)
    rows = counter.values_range(3, counter.STREAM_ROWS, 0, N * D, counter.KIND_DYADIC).reshape(N, D)
    tokens = np.array([9, 8, 9])
    w, _, _ = oracle.token_weights(tokens, 9, 3)
    res = _run_sparse(ids.astype(np.int64), rows, off, w, tokens, 9, 3, R, plan=plan)
    _check_sparse(res, ids, rows, off, w, tokens, 9, 3, expect_exact=True)


@pytest.mark.parametrize("opt,decay", [("adagrad", "token"), ("adagrad", "id_tag"), ("adam", "id_tag")])
@pytest.mark.parametrize("D", [4, 12, 16, 28, 128, 256])
def test_fused_apply_at_the_other_widths(D, opt, decay):
    """The row pass applies the rows at every number of lanes per row (one to
    64 groups per wave share a ring of finished segments; rows that are not
    whole 64-byte pieces go through the caches): table, state, tags and counts are bitwise those of the aggregation and the row apply as two calls.
    Few long segments and many short ones, so that the ring fills unevenly."""
    K, R = 9, 30_000
    rng = np.random.default_rng(D)
    sizes = rng.integers(0, 5_000, K)
    N = int(sizes.sum())
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    ids = np.where(rng.random(N) < 0.3, rng.integers(0, 3, N), rng.integers(0, R, N)).astype(np.int64)
    rows = counter.values_range(D, counter.STREAM_ROWS, 0, N * D, counter.KIND_GRAD,
                                counter.grad_scale(1e-2)).reshape(N, D)
    step, iota = 1000, 3
    tokens = step - rng.integers(0, 6, K)
    tag = workload.tag_values(5, np.arange(R), step)
    w, _, _ = oracle.token_weights(tokens, step, iota)
    table0, slots0 = _table_and_state(R, D, opt, 5)
    d_in = (dev(ids), dev(rows), dev(off), dev(w), dev(tokens))
    sep = _sparse_step(*d_in, step, iota, R, tag, decay, opt, False, True, table0, slots0)
    fus = _sparse_step(*d_in, step, iota, R, tag, decay, opt, True, False, table0, slots0)
    assert sep["err"] == 0 and fus["err"] == 0
    U = int(sep["num_unique"][0])
    assert int(fus["num_unique"][0]) == U
    for k in ("unique_ids", "contrib_count", "active_count"):
        assert_exact(fus[k][:U], sep[k][:U], k)
    assert torch.equal(fus["table"], sep["table"])
    assert all(torch.equal(a, b) for a, b in zip(fus["slots"], sep["slots"]))
    if decay == "id_tag":
        assert_exact(fus["tag"], sep["tag"], "tag")


@pytest.mark.parametrize("plan", [gba.SORT_PLAIN, gba.SORT_HOT])
@pytest.mark.parametrize("R", [200, 70_000])
@pytest.mark.parametrize("N", [1, 6, 1027, 40_001])
def test_fractional_weights_at_the_ends_of_the_input(N, R, plan):
    """Weights other than 0 and 1 go from the position pass to the row pass
    through an array of the sort (one pass at R = 200, three at 70,000): inputs
    that end inside a lane's four positions, with 0, 1 and fractions side by
    side, some batches without any fraction."""
    K, D = 8, 8
    rng = np.random.default_rng(N + R)
    ids = rng.integers(0, R, N).astype(np.int64)
    ids[rng.random(N) < 0.2] = R // 2
    cut = np.sort(rng.integers(0, N + 1, K - 1))
    off = np.concatenate([[0], cut, [N]]).astype(np.int64)
    rows = counter.values_range(N, counter.STREAM_ROWS, 0, N * D, counter.KIND_DYADIC).reshape(N, D)
    tokens = np.full(K, 10)
    w = np.array([1.0, 0.5, 0.0, 1.0, 0.25, 0.0, 1.0, 0.75], np.float32)
    res = _run_sparse(ids, rows, off, w, tokens, 10, 2, R, plan=plan)
    _check_sparse(res, ids, rows, off, w, tokens, 10, 2, expect_exact=True)


@pytest.mark.parametrize("D", [4, 32, 64])
@pytest.mark.parametrize("opt", ["adagrad", "adam"])
def test_offsets_out_of_order(opt, D):
    """Offsets that go up and down are reported; a segment may then change its
    contribution more often than there are contributions, past the row pass's
    table of reciprocals."""
    K, R, N = 200, 1_000, 40_000
    rng = np.random.default_rng(D)
    off = rng.integers(0, N + 1, K + 1)
    off[0], off[K] = 0, N
    ids = np.where(rng.random(N) < 0.5, 5, rng.integers(0, R, N)).astype(np.int64)
    rows = np.zeros((N, D), np.float32)
    tokens = np.full(K, 1000)
    table0, slots0 = _table_and_state(R, D, opt, 5)
    out = _sparse_step(dev(ids), dev(rows), dev(off.astype(np.int64)), dev(np.ones(K, np.float32)), dev(tokens), 1000, 3,
                       R, None, "token", opt, True, True, table0, slots0)
    assert out["err"] == gba.DERR_OFFSETS
    assert int(out["num_unique"][0]) == np.unique(ids).size
