"""Setting the knobs a context has, and tuning it for one batch size, keep the launches that calls with few
members share; a knob below the default narrows them, and the default brings them back."""
import pytest

from paper_2207_04620_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule", [15, 0])
@pytest.mark.parametrize("members", [1, 3])
def test_knobs_keep_the_launches_of_few_members(schedule, members):
    import torch
    assert torch.cuda.is_available()
    from paper_2207_04620_amd import he
    ctx = he.Context(I.small(log_n=12, n_q=7, alpha=2, q_bits=40, p_bits=50), schedule=schedule, h_list=[16])
    pairs = [[ctx.encrypt(m.ravel(), nonce=2 * i + k) for k, m in enumerate(I.matrix_pair(80 + i, 16))]
             for i in range(members)]

    def launches():
        ctx.profile(True)
        ctx.matmul_batch([p[0] for p in pairs], [p[1] for p in pairs], [16] * members)
        ctx.sync()
        ctx.profile(False)
        return sum(k["launches"] for k in ctx.profile_report().values())

    def narrower(rep):
        """the tuner took a knob below the default, which then has to be faster than the first candidate"""
        first, best = rep["candidates"][0], rep["chosen"]
        assert first["pair_batch"] == 4 and first["max_group"] == min(32, batch)
        took = next(c for c in rep["candidates"] if all(c[k] == best[k] for k in ("pair_batch", "max_group", "overlap")))
        return best["pair_batch"] < 4 and took["ms"] < 0.99 * first["ms"]

    default = launches()
    knobs = ctx.tuning()
    ctx.set_tuning(**knobs)
    assert launches() == default
    ctx.set_tuning(2, 32)
    assert launches() > default
    ctx.set_tuning(8, 32)
    assert launches() <= default
    ctx.set_tuning(**knobs)
    assert launches() == default
    for batch in (members, 16):
        rep = ctx.autotune(16, 5, batch)
        assert ctx.tuning() == rep["chosen"]
        assert rep["source"] != "timed" or rep["chosen"]["pair_batch"] >= 4 or narrower(rep)
        if ctx.tuning()["pair_batch"] >= 4 and ctx.tuning()["overlap"] == 0:
            ctx.set_tuning(ctx.tuning()["pair_batch"], 32)
            assert launches() <= default
        ctx.set_tuning(**knobs)
    ctx.close()
