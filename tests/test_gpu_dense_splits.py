"""The dense calls at sizes that take each number of vectors per thread (1 to
4 where four for every thread would leave part of the chip idle, else 4 to 16;
which one also depends on the number of gradients), with whole, ragged and
scalar ends: the sum bit for bit, and the fused, separate and early forms
bitwise equal."""
import pytest
import torch

import paper_2205_11048_amd as gba

pytestmark = pytest.mark.gpu
DEV = "cuda"
LR, EPS, B1, B2, T = 0.01, 1e-8, 0.9, 0.999, 7

# with 256 compute units of 512 threads, vectors per thread for 3 and for 40
# gradients: 1 1 1 1 4 6 4 10 4 4 4 12 10 and 1 2 3 4 4 6 4 10 12 14 16 12 10
# (two or more steps per compute unit in the last two); the early form's
# folds (2, 1 and 38 gradients) and its finishing call have their own rules
SIZES = [100_003, 1_000_003, 1_500_001, 2_000_002, 2_097_152, 3_000_001, 4_194_304, 5_200_003, 6_000_001, 7_300_002,
         8_000_003, 16_777_217, 20_000_001]


@pytest.mark.parametrize("K", [3, 40])
@pytest.mark.parametrize("P", SIZES)
def test_dense_vectors_per_thread(P, K):
    gen = torch.Generator(device=DEV).manual_seed(P)
    grads = [torch.empty(P, device=DEV).normal_(0, 1e-2, generator=gen) for _ in range(3)]
    grads[1].fill_(float("nan"))                               # excluded: never read
    w = torch.tensor([1.0, 0.0, 0.5] + [0.0] * (K - 3), device=DEV)
    table = gba.pointer_table(grads + [grads[1]] * (K - 3))
    ref = ((grads[0].double() + 0.5 * grads[2].double()) / K).float()
    out = torch.full((P,), 7.0, device=DEV)
    gba.gba_aggregate_dense(table, w, P, out)
    assert torch.equal(out, ref)

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


@pytest.mark.parametrize("opt", [gba.DENSE_SUM, gba.DENSE_ADAGRAD, gba.DENSE_ADAM])
@pytest.mark.parametrize("P", [40_000_000, 64_000_000, 72_000_000, 90_000_000, 98_500_000, 200_000_000])
def test_large_sums_keep_long_runs(P, opt):
    """Where fewer vectors per thread than 16 would save a sixteenth of the
    block steps or less, the shorter runs cost more: one launch per 256 steps
    of 32,768 elements, the blocks the GPU holds at once."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the counts are those of 256 compute units")
    assert gba.gba_aggregate_dense_launches(P, 64, opt) == -(-P // (256 * 32_768))
