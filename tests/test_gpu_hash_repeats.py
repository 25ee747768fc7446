"""Find-or-insert where IDs repeat inside a wave: one lane asks for the slot
and the row of all lanes that hold its ID, whether the ID is among a wave's
first distinct values or past the ones looked at; every position of an ID gets
one row, rows are handed out once each, and a full pool serves the rest later."""
import pytest
import torch

import paper_2205_11048_amd as gba

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _ids(kind, n, g):
    i = torch.arange(n, device=DEV)
    if kind == "one":
        return torch.full((n,), 12345, dtype=torch.int64, device=DEV)
    if kind == "pairs":                       # 32 distinct IDs per wave, each twice, half a wave apart
        return (i // 64) * 32 + i % 32
    if kind == "late":                        # 40 distinct IDs, then one ID to the wave's end
        return torch.where(i % 64 < 40, 10 + i, 7)
    return (torch.rand(n, device=DEV, generator=g).pow(6) * 50_000).to(torch.int64)


@pytest.mark.parametrize("capacity_log2", [12, 18])
@pytest.mark.parametrize("kind", ["one", "pairs", "late", "skewed"])
@pytest.mark.parametrize("n", [1, 63, 257, 2_000, 200_001])
def test_repeated_ids_on_an_empty_index(n, kind, capacity_log2):
    g = torch.Generator(device=DEV).manual_seed(n)
    ids = _ids(kind, n, g) * -7046029254386353131 + 5      # over the whole 64-bit range
    unique = torch.unique(ids)
    U = unique.numel()
    cap = 1 << capacity_log2
    if U > cap // 2:
        cap = 1 << (2 * U).bit_length()
    slot_ids = torch.empty(cap, dtype=torch.int64, device=DEV)
    slot_rows = torch.empty(cap, dtype=torch.int32, device=DEV)
    gba.gba_hash_clear(slot_ids, slot_rows)
    rows = torch.full((n,), -5, dtype=torch.int64, device=DEV)
    num_rows = torch.zeros(1, dtype=torch.int64, device=DEV)
    num_new = torch.zeros(1, dtype=torch.int64, device=DEV)
    row_ids = torch.full((U + 3,), -5, dtype=torch.int64, device=DEV)
    ws = torch.empty(gba.gba_hash_workspace_size(n), dtype=torch.uint8, device=DEV)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    small = U // 2                                         # a pool for half of the IDs, then for all
    if small:
        gba.gba_hash_find_or_insert(slot_ids, slot_rows, ids, rows, num_rows, small, ws, row_ids, num_new, err)
        assert int(num_rows.item()) == small and int(num_new.item()) == U
        assert int(err.item()) == gba.DERR_TABLE_FULL
        served = rows >= 0
        assert torch.equal(row_ids[rows[served]], ids[served])
        assert torch.unique(ids[served]).numel() == small
        err.zero_()
    gba.gba_hash_find_or_insert(slot_ids, slot_rows, ids, rows, num_rows, U + 3, ws, row_ids, num_new, err)
    assert int(err.item()) == 0
    assert int(num_rows.item()) == U and int(num_new.item()) == U - small
    assert torch.equal(row_ids[rows], ids) and torch.equal(torch.unique(rows), torch.arange(U, device=DEV))
    again = torch.full((n,), -5, dtype=torch.int64, device=DEV)
    gba.gba_hash_find_or_insert(slot_ids, slot_rows, ids, again, num_rows, U + 3, ws, row_ids, num_new, err)
    assert torch.equal(again, rows) and int(num_new.item()) == 0 and int(num_rows.item()) == U
