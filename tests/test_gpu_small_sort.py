"""The plain ID sort at the edges of its rules: one launch per pass up to
32,768 keys, two below 2^20 (2^21 to 2^22 for keys that 9-bit digits take in a
pass less), three above, the sizes up to which digits of 10 and 11 bits save a
pass, tiles of 2048 and 4096 keys; against a stable sort, which the outputs
equal element for element."""
import pytest
import torch

import paper_2205_11048_amd as gba

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _sort(ids, R, plan=gba.SORT_PLAIN):
    n = ids.numel()
    keys = torch.full((n,), -5, dtype=torch.int32, device=DEV)
    index = torch.full((n,), -5, dtype=torch.int32, device=DEV)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = torch.empty(gba.gba_sort_ids_workspace_size(n, R, plan), dtype=torch.uint8, device=DEV)
    gba.gba_sort_ids(ids, R, keys, index, ws, plan, err)
    return keys.to(torch.int64) & 0xFFFFFFFF, index.to(torch.int64), int(err.item())


def _ids(n, R, seed, skew):
    g = torch.Generator(device=DEV).manual_seed(seed)
    u = torch.rand(n, device=DEV, dtype=torch.float64, generator=g)
    ids = (u.pow(skew) * R).to(torch.int64).clamp_(max=R - 1)
    return (ids * 2654435761 + 977) % R      # hot IDs apart from one another


@pytest.mark.parametrize("R", [1, 2, 200, 256, 1000, 2047, 4096, 100_000, 1 << 20, 1_234_567, 1 << 22, 10_000_000,
                               100_000_000, 1 << 29, (1 << 31) - 1, 1 << 32])
@pytest.mark.parametrize("n", [1, 63, 2047, 2048, 2049, 4097, 32_767, 32_768, 32_769, 100_003])
def test_sort_key_widths(n, R):
    ids = _ids(n, R, n + R % 1009, 4.0)
    keys, index, err = _sort(ids, R)
    ref, ref_index = torch.sort(ids, stable=True)
    assert err == 0
    assert torch.equal(keys, ref) and torch.equal(index, ref_index)


@pytest.mark.parametrize("R", [500, 200_000, 3_000_000, 30_000_000, 1 << 32])
@pytest.mark.parametrize("n", [(1 << 19) - 1, 1 << 19, (1 << 20) - 1, 1 << 20, (1 << 21) + 1, (1 << 22) - 1])
def test_sort_digit_and_tile_rules(n, R):
    ids = _ids(n, R, n % 1013, 3.0)
    keys, index, err = _sort(ids, R)
    ref, ref_index = torch.sort(ids, stable=True)
    assert err == 0
    assert torch.equal(keys, ref) and torch.equal(index, ref_index)


@pytest.mark.parametrize("bits", [9, 10, 11, 17, 18, 20, 22, 25, 27, 30, 32])
@pytest.mark.parametrize("n", [(3 << 16) - 1, 3 << 16, (5 << 16) - 1, 5 << 16, (1 << 20) + 1, (1 << 21) - 1, 1 << 21,
                               (3 << 20) - 1, 3 << 20, (1 << 22) - 1])
def test_sort_digit_lines(n, bits):
    R = 1 << bits
    ids = _ids(n, R, n % 1013 + bits, 3.0)
    keys, index, err = _sort(ids, R)
    ref, ref_index = torch.sort(ids, stable=True)
    assert err == 0
    assert torch.equal(keys, ref) and torch.equal(index, ref_index)


@pytest.mark.parametrize("n", [30_000, 250_000, 1_100_000])
def test_sort_one_id_and_bad_ids(n):
    """Every key in one bin, and IDs outside [0, R), which are reported and sorted as 0."""
    R = 5_000_000
    keys, index, err = _sort(torch.full((n,), 4_321_987, dtype=torch.int64, device=DEV), R)
    assert err == 0 and bool((keys == 4_321_987).all())
    assert torch.equal(index, torch.arange(n, device=DEV))
    ids = _ids(n, R, 3, 1.0)
    ids[7], ids[n // 2], ids[n - 1] = -1, R, 1 << 40
    keys, index, err = _sort(ids, R)
    assert err == gba.DERR_ID_RANGE
    ids[7] = ids[n // 2] = ids[n - 1] = 0
    ref, ref_index = torch.sort(ids, stable=True)
    assert torch.equal(keys, ref) and torch.equal(index, ref_index)
