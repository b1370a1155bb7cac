"""A caller's device allocator with a byte budget: a call whose wide launches do not fit it falls back to the
narrow ones with the same results, a batch's side-stream blocks do not starve the call after it, blocks
come back drained (the allocator hands a returned block out again at once), and all of them come back."""
import ctypes as C

import numpy as np
import pytest

from paper_2207_04620_amd import inputs as I

pytestmark = pytest.mark.gpu


class Arena:
    """first fit in one tensor; at most 'budget' bytes handed out"""

    def __init__(self, he, nbytes):
        import torch
        self.mem = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        self.base, self.size, self.used, self.budget, self.refused = self.mem.data_ptr(), nbytes, {}, nbytes, 0
        self.calls = (C.CFUNCTYPE(C.c_void_p, C.c_size_t, C.c_void_p)(self.alloc),
                      C.CFUNCTYPE(None, C.c_void_p, C.c_void_p)(self.free))
        dev, (a, f) = he._Device, self.calls
        self.device = lambda stream, *_: dev(stream, C.cast(a, C.c_void_p), C.cast(f, C.c_void_p), None)

    def alloc(self, n, _):
        at = 0
        for p in sorted(self.used):
            if p - at >= n:
                break
            at = p + self.used[p]
        if sum(self.used.values()) + n > self.budget or at + n > self.size:
            self.refused += 1
            return None
        self.used[at] = n
        return self.base + at

    def free(self, p, _):
        del self.used[p - self.base]


PRM = I.small(log_n=12, n_q=6, alpha=2, q_bits=40, p_bits=50)


def _operands(ctx, count):
    return [[ctx.encrypt(m.ravel(), nonce=2 * i + k) for k, m in enumerate(I.matrix_pair(90 + i, 16))]
            for i in range(count)]


def _peak(ctx, call):
    before, _ = ctx.pool_stats(reset=True)
    keep = call()  # noqa: F841 (the result counts)
    ctx.sync()
    return ctx.pool_stats()[1] - before


@pytest.mark.parametrize("schedule", [15, 0])
@pytest.mark.parametrize("mixed_first", [False, True])
def test_wide_call_falls_back_to_narrow(schedule, mixed_first, monkeypatch):
    import torch
    assert torch.cuda.is_available()
    from paper_2207_04620_amd import he

    def batch(ctx, ops):
        return ctx.matmul_batch([ops[0][0], ctx.drop(ops[1][0], 4)], [ops[0][1], ops[1][1]], [16, 16])

    plain = he.Context(PRM, schedule=schedule, h_list=[16])
    ops = _operands(plain, 2)
    single = lambda c, o: c.matmul(o[0][0], o[0][1], 16)  # noqa: E731
    plain.counters(reset=True)
    want, counts = plain.export(single(plain, ops)), plain.counters()
    want_batch = [plain.export(c) for c in batch(plain, ops)]
    wide = _peak(plain, lambda: single(plain, ops))
    plain.pool_limit(1 << 40)
    narrow = _peak(plain, lambda: single(plain, ops))
    plain.close()
    assert narrow < wide

    arena = Arena(he, 4 << 30)
    monkeypatch.setattr(he, "_Device", arena.device)
    ctx = he.Context(PRM, schedule=schedule, h_list=[16])
    ops = _operands(ctx, 2)
    if mixed_first:
        assert all(np.array_equal(ctx.export(c), w) for c, w in zip(batch(ctx, ops), want_batch))
    ctx.sync()
    in_use, _ = ctx.pool_stats()
    arena.budget = in_use + (narrow + wide) // 2
    for _ in range(3):
        arena.refused = 0
        ctx.counters(reset=True)
        assert np.array_equal(ctx.export(single(ctx, ops)), want) and ctx.counters() == counts
        assert arena.refused > 0 or mixed_first
    ctx.pool_limit(1)  # the cached blocks go back
    ctx.pool_limit(0)
    assert sum(arena.used.values()) == ctx.pool_stats()[0]
    arena.budget = in_use  # not even the narrow call fits: refused, and the context goes on
    with pytest.raises(he.HEError, match="HE_ENOMEM") as e:
        single(ctx, ops)
    del e  # its traceback holds the operands
    arena.budget = arena.size
    assert np.array_equal(ctx.export(single(ctx, ops)), want)
    ops = None
    ctx.close()
    assert not arena.used
