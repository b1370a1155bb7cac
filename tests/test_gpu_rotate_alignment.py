"""he_rotate_noalloc into a result buffer at an odd multiple of 8 bytes: the residues of he_rotate, and
not a word outside the buffer."""
import numpy as np
import pytest

from paper_2207_04620_amd import inputs as I

pytestmark = pytest.mark.gpu


# a ring below one row of 2048 words, one of a single row, and two with both passes (the second in several digits)
@pytest.mark.parametrize("log_n,n_q,alpha,level", [(9, 3, 3, 2), (11, 4, 2, 3), (12, 6, 2, 0), (12, 6, 2, 5)])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_result_at_any_word(log_n, n_q, alpha, level, shift):
    import torch
    assert torch.cuda.is_available()
    from paper_2207_04620_amd import he
    ctx = he.Context(I.small(log_n=log_n, n_q=n_q, alpha=alpha, q_bits=40, p_bits=50), h_list=[],
                     stream=torch.cuda.current_stream().cuda_stream)
    ctx.gen_rotation_key(3)
    x = ctx.encrypt(np.linspace(-1, 1, ctx.n // 2), level=level, nonce=4)
    want, nl = ctx.export(ctx.rotate(x, 3)), level + 1
    mods = [i for _ in range(2) for i in range(nl)]
    inp = torch.from_numpy(ctx.export(x).reshape(-1, ctx.n).view(np.int64)).cuda()
    ctx.ntt(inp, mods)
    words = inp.numel()
    buf = torch.full((words + 8,), -7, dtype=torch.int64, device="cuda")
    assert buf.data_ptr() % 16 == 0
    ctx.rotate_noalloc(inp.data_ptr(), level, 3, buf.data_ptr() + 8 * shift)
    ctx.sync()
    got = buf[shift:shift + words].clone().view(-1, ctx.n)
    assert (buf[:shift] == -7).all() and (buf[shift + words:] == -7).all()
    ctx.ntt(got, mods, inverse=True)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy().view(np.uint64).reshape(want.shape), want)
    ctx.close()
