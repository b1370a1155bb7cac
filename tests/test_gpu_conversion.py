"""Key switching and rescaling through the matrix-unit base conversion, bit-exact against the oracle.

Each case is a ring and chain at an edge of the conversion: one to five column stages (and six, where the
separate passes run), one to eight sources per digit and special primes, targets of both kinds
alone, in full sets of four and with a remainder, primes just below and above 2^46, and small ones.
"""
import numpy as np
import pytest

import oracle as O
from paper_2207_04620_amd import inputs as I

pytestmark = pytest.mark.gpu

# (log_n, Q bits, P bits, alpha, levels)
CASES = [
    (12, [60] + [45] * 7, [60] * 5, 5, (7, 4, 1)),        # one column stage, five sources
    (12, [40, 30, 30, 30], [40], 1, (3, 1)),              # small primes, one source, FP64 everywhere
    (13, [60] * 3 + [30] * 7, [60] * 8, 8, (9, 8, 2)),    # two stages, eight sources
    (14, [60] + [45] * 6, [60] * 5, 5, (6, 3)),           # three stages, the shared fifth source
    (14, [50, 46, 47, 46, 45, 44, 43], [60] * 6, 6, (6, 5)),  # primes about 2^43 and 2^46, six sources
    (14, [60] * 6, [60] * 7, 7, (5, 1)),                  # integer targets only, seven sources
    (15, [60] + [45] * 5, [60] * 4, 3, (5, 4, 2)),        # four stages, up to four sources
    (15, [60] + [45] * 9, [60, 60, 60, 56, 45], 5, (9, 6, 5)),
    (15, [46] * 8, [47] * 6, 6, (7, 6)),
    (15, [60] * 2 + [45] * 7, [60] * 8, 8, (8, 7)),
    (16, [60] + [45] * 6, [60] * 5, 6, (6, 2)),           # five stages, one member: the rescale alone
    (16, [60] + [45] * 7, [60] * 7, 7, (7,)),             # five stages, seven sources
    (17, [60, 45, 45], [60, 60], 2, (2, 1)),              # six stages: separate passes
]


@pytest.mark.parametrize("log_n,q_bits,p_bits,alpha,levels", CASES)
def test_conversion_edges(log_n, q_bits, p_bits, alpha, levels):
    import torch  # its HIP runtime, before the library's
    assert torch.cuda.is_available()
    from paper_2207_04620_amd import he
    prm = I.Params("conv", log_n, q_bits, p_bits, alpha, 30.0, 17 + log_n, [])
    print(f"[conversion] N=2^{log_n} Q={q_bits} P={p_bits} alpha={alpha}", flush=True)
    g, o = he.Context(prm, h_list=[]), O.Ctx.from_params(prm)

    def same(x, y):
        assert np.array_equal(g.export(x), y.export())

    z, w = I.matrix_pair(log_n, 8)
    g.gen_rotation_key(3)
    for lv in levels:
        ga, gb = g.encrypt(z.ravel(), level=lv, nonce=1), g.encrypt(w.ravel(), level=lv, nonce=2)
        oa, ob = o.encrypt(z.ravel(), level=lv, nonce=1), o.encrypt(w.ravel(), level=lv, nonce=2)
        gt, ot = g.tensor(ga, gb), o.tensor(oa, ob)
        gm, om = g.relin(gt), o.relin(ot)
        same(gm, om)
        same(g.rescale(gm), o.rescale(om))
        same(g.rescale(gt), o.rescale(ot))  # three polynomials
        same(g.rotate(ga, 3), o.rotate(oa, 3))
    g.close()


@pytest.mark.parametrize("p_count,alpha", [(4, 4), (5, 6), (6, 5)])
def test_five_stages_of_several_members(p_count, alpha):
    """N = 2^16, eight members a launch: ModUp and ModDown as one column pass"""
    import torch
    assert torch.cuda.is_available()
    from paper_2207_04620_amd import he
    prm = I.Params("conv16", 16, [60] + [45] * 6, [60] * p_count, alpha, 40.0, 5, [])
    g, o = he.Context(prm, h_list=[]), O.Ctx.from_params(prm)
    xs = [I.sign_inputs(3 + i, 1, 16)[0].ravel() for i in range(8)]
    ys = g.sign_approx_batch([g.encrypt(x, nonce=1 + i) for i, x in enumerate(xs)], 1, 1, 0)
    for i in (0, 7):
        oy = o.sign(o.encrypt(xs[i], nonce=1 + i), 1, 1, relu=False)
        assert np.array_equal(g.export(ys[i]), oy.export()) and ys[i].scale == oy.scale
    g.close()
