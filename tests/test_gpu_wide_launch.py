"""Direct calls with few members take more rotation sets per launch than the knob's default; the
results and the operation counts are those of every setting, also under a capped allocation cache."""
import numpy as np
import pytest

from paper_2207_04620_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule", [15, 2, 0, 3, 4, 5, 8, 10])
@pytest.mark.parametrize("members", [1, 2, 3, 5, 8, 16])
def test_default_equals_every_setting(schedule, members):
    import torch
    assert torch.cuda.is_available()
    from paper_2207_04620_amd import he
    ctx = he.Context(I.small(log_n=12, n_q=6, alpha=2, q_bits=40, p_bits=50), schedule=schedule, h_list=[16])
    pairs = [[ctx.encrypt(m.ravel(), nonce=2 * i + k) for k, m in enumerate(I.matrix_pair(80 + i, 16))]
             for i in range(members)]
    As, Bs = [p[0] for p in pairs], [p[1] for p in pairs]

    def product():
        ctx.counters(reset=True)
        res = [ctx.export(c) for c in ctx.matmul_batch(As, Bs, [16] * members)]
        res += [ctx.export(c) for c in ctx.transpose_batch(As, 16)]
        res += [ctx.export(c) for c in ctx.matmul_batch_ex(As, Bs, [(16, 4, 2)] * members)]
        return res, ctx.counters()

    ref, counts = product()
    ref, counts = product()  # keys and masks exist
    in_use, _ = ctx.pool_stats()
    ctx.pool_limit(in_use + (1 << 31))  # a cap keeps the knob's sets per launch
    got, again = product()
    ctx.pool_limit(0)
    assert again == counts and all(np.array_equal(x, y) for x, y in zip(got, ref))
    for sets in (1, 4, 16):
        ctx.set_tuning(sets, 32)
        got, again = product()
        assert again == counts and all(np.array_equal(x, y) for x, y in zip(got, ref)), sets
    ctx.close()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("d", [1, 2, 3, 4, 6, 7])
@pytest.mark.parametrize("members", [1, 3, 33])
def test_polynomial_levels_equal_terms(d, mode, members):
    """a level of g_d in one pass against term by term (under a cap): limbs, scales and counts"""
    import torch
    assert torch.cuda.is_available()
    from paper_2207_04620_amd import he
    ctx = he.Context(I.small(log_n=12, n_q=10, alpha=2, q_bits=40, p_bits=50))
    xs = [ctx.encrypt(I.sign_inputs(7 + i, 1, 16)[0].ravel(), nonce=i) for i in range(members)]

    def evaluate():
        ctx.counters(reset=True)
        ys = ctx.sign_approx_batch(xs, d, 2, mode)
        return [(ctx.export(y), y.scale, y.level) for y in ys], ctx.counters()

    ref, counts = evaluate()
    in_use, _ = ctx.pool_stats()
    ctx.pool_limit(in_use + (1 << 31))
    got, again = evaluate()
    ctx.pool_limit(0)
    assert again == counts
    for (x, s, l), (y, t, m) in zip(got, ref):
        assert np.array_equal(x, y) and s == t and l == m
    ctx.close()
