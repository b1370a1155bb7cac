"""A sign evaluation under a cap takes the memory of its largest step and no more."""
import pytest

from paper_2207_04620_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("members", [1, 3])
def test_peak_of_a_capped_evaluation(members):
    import torch
    assert torch.cuda.is_available()
    from paper_2207_04620_amd import he
    prm = I.small(log_n=12, n_q=8, alpha=2, q_bits=40, p_bits=50)
    ctx = he.Context(prm)
    xs = [ctx.encrypt(I.sign_inputs(3 + i, 1, 16)[0].ravel(), nonce=i) for i in range(members)]
    # the first product of g_3's x^7: beside x, x^2 and x^4, the sum so far and the multiple of x, it holds the tensor
    # product, its lift, the result, the inner product over Q_l and P and the converted limbs (limbs per member)
    l, k = prm.max_level, len(prm.p_bits)  # x has l + 1 limbs, the product l
    beta = -(-l // prm.alpha)
    words = 2 * (l + 1) + 2 * l + 2 * (l - 1) + 2 * l + 2 * l + 3 * l + beta * (l + k) + 2 * l + 2 * (l + k) + 2 * l
    for _ in range(2):  # (the keys exist the second time)
        ctx.pool_limit(1 << 40)
        before, _ = ctx.pool_stats(reset=True)
        ctx.sign_approx_batch(xs, 3, 2)
        ctx.sync()
        peak = ctx.pool_stats()[1] - before
    assert peak <= 8 * ctx.n * members * words, (peak / (8 * ctx.n * members), words)
    ctx.pool_limit(before + 8 * ctx.n * members * words)
    ctx.sign_approx_batch(xs, 3, 2)
    ctx.close()
