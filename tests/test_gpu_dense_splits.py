"""The dense calls at sizes that take each number of vectors per thread (1 to
4 where four for every thread would leave part of the chip idle, else 4 to
16), with whole, ragged and scalar ends: the sum bit for bit, and the fused,
separate and early forms bitwise equal."""
import pytest
import torch

import paper_2205_11048_amd as gba

pytestmark = pytest.mark.gpu
DEV = "cuda"
LR, EPS, B1, B2, T = 0.01, 1e-8, 0.9, 0.999, 7

# with 256 compute units of 512 threads: vectors per thread 1, 2, 3, 4, 4, 6, 4, 10, 12, 14, 16, and two or more
# steps per compute unit (10 and 16)
SIZES = [100_003, 1_000_003, 1_500_001, 2_000_002, 2_097_152, 3_000_001, 4_194_304, 5_200_003, 6_000_001, 7_300_002,
         8_000_003, 16_777_217, 20_000_001]


@pytest.mark.parametrize("P", SIZES)
def test_dense_vectors_per_thread(P):
    K = 3
    gen = torch.Generator(device=DEV).manual_seed(P)
    grads = [torch.empty(P, device=DEV).normal_(0, 1e-2, generator=gen) for _ in range(K)]
    grads[1].fill_(float("nan"))                               # excluded: never read
    w = torch.tensor([1.0, 0.0, 0.5], device=DEV)
    table = gba.pointer_table(grads)
    ref = ((grads[0].double() + 0.5 * grads[2].double()) / K).float()
    out = torch.full((P,), 7.0, device=DEV)
    gba.gba_aggregate_dense(table, w, P, out)
    assert torch.equal(out, ref)
    del grads[1]

    def state():
        g = torch.Generator(device=DEV).manual_seed(5)
        return [torch.empty(P, device=DEV).uniform_(0.1, 0.3, generator=g) for _ in range(3)]

    p, a, _ = state()
    gba.gba_apply_adagrad(p, a, out, LR, EPS)
    fp, fa, _ = state()
    gba.gba_aggregate_apply_dense_adagrad(table, w, P, fp, fa, LR, EPS)
    assert torch.equal(fp, p) and torch.equal(fa, a)
    ep, ea, _ = state()
    run = torch.zeros(P, dtype=torch.float64, device=DEV)
    gba.gba_accumulate_dense(table[:2], w[:2], P, run)
    gba.gba_accumulate_dense(table[2:], w[2:], P, run)
    gba.gba_finalize_apply_dense_adagrad(run, K, P, ep, ea, LR, EPS)
    assert torch.equal(ep, p) and torch.equal(ea, a) and not bool(run.any())

    p, m, v = state()
    gba.gba_apply_adam(p, m, v, out, LR, B1, B2, EPS, T)
    fp, fm, fv = state()
    g_bar = torch.full((P,), 7.0, device=DEV)
    gba.gba_aggregate_apply_dense_adam(table, w, P, fp, fm, fv, LR, B1, B2, EPS, T, out=g_bar)
    assert torch.equal(g_bar, ref)
    assert torch.equal(fp, p) and torch.equal(fm, m) and torch.equal(fv, v)
