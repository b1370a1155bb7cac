"""Encoding and decoding on the device: the integers of the oracle's 113-bit encoder, bit for bit, over the
ranges its fixed point takes and at their edges, and decryption against the oracle's integers."""
import numpy as np
import pytest

import oracle as O
from paper_2207_04620_amd import inputs as I

pytestmark = pytest.mark.gpu


def _pair(log_n):
    import torch  # its HIP runtime, before the library's
    assert torch.cuda.is_available()
    from paper_2207_04620_amd import he
    prm = I.Params("enc", log_n, [60, 45, 40], [60], 3, 40.0, 5, [])
    return he.Context(prm, h_list=[]), O.Ctx.from_params(prm), he


def _values(log_n):
    rng = np.random.default_rng(log_n)
    half = 1 << (log_n - 1)
    wide = rng.uniform(-1, 1, half) * 2.0 ** rng.integers(-40, 1, half)
    mixed = np.where(np.arange(half) % 7 == 0, 1e-300, rng.uniform(-1, 1, half))
    mixed[1], mixed[2], mixed[3] = 5e-324, -0.0, -1e-310
    return [(rng.uniform(-1, 1, half), 40), (rng.uniform(-1, 1, 16), 45), (wide, 60), (mixed, 30), (np.array([0.7]), 61),
            (np.zeros(4), 40), (np.array([-3.0e5, 1.0]), 20), (rng.uniform(-1, 1, half) * 1e-9, 20),
            (rng.uniform(-1, 1, 8) * 2.0 ** 900, -870), (rng.uniform(-1, 1, 8) * 1e-290, 990),
            (np.array([1.0, -0.3]), 61.4), (np.array([0.99, 0.3]), 62.5)]  # the last is above 2^62


@pytest.mark.parametrize("log_n", [8, 9, 11, 12, 15, 16])
def test_encode_edges(log_n):
    g, o, _ = _pair(log_n)
    for i, (v, log_scale) in enumerate(_values(log_n)):
        scale = float(2.0 ** log_scale)
        a, (b, tie) = g.encode(v, scale), o.encode(v, scale)
        print(f"[encode] N=2^{log_n} case {i} tie {tie:.1e}", flush=True)
        # (an exact zero is half a unit from a tie)
        assert tie > 1e-12
        assert np.array_equal(a, b), f"case {i}: {np.flatnonzero(a != b)[:4]}"
    g.close()


@pytest.mark.parametrize("log_n,level", [(8, 0), (9, 1), (12, 2), (15, 2), (15, 0)])
def test_decrypt_matches_oracle(log_n, level):
    g, o, he = _pair(log_n)
    rng = np.random.default_rng(level)
    z = rng.uniform(-1, 1, g.n // 2)
    gc, oc = g.encrypt(z, level=level, nonce=4), o.encrypt(z, level=level, nonce=4)
    assert np.array_equal(g.export(gc), oc.export())
    m = o.decrypt_coeffs(oc)
    assert np.array_equal(g.decrypt_coeffs(gc), m)
    # both transforms: N terms, each through log2 N + 2 rounded complex operations
    tol = 8 * (log_n + 2) * 2.0 ** -52 * np.abs(m).sum() / g.scale
    for n in (g.n // 2, 5):
        assert np.abs(g.decrypt(gc, n) - o.decrypt(oc, n)).max() <= tol
    # a degree-2 ciphertext, and plaintexts up to q_0 q_1 / 2 with both signs
    if level:
        t, u = g.tensor(gc, gc), o.tensor(oc, oc)
        assert np.array_equal(g.decrypt_coeffs(t), o.decrypt_coeffs(u))
        q0, q1 = g.moduli[0], g.moduli[1]
        half = q0 * q1 // 2
        w = [int(x) for x in rng.integers(-2 ** 62, 2 ** 62, g.n)]
        w = [(x * (half >> 62)) for x in w]
        w[:6] = [half, -half, half - 1, 2 ** 64, -2 ** 64 - 1, 2 ** 53 + 1]
        arr = np.zeros((2, level + 1, g.n), np.uint64)
        for i in range(level + 1):
            arr[0, i] = np.array([x % g.moduli[i] for x in w], np.uint64)
        assert np.array_equal(g.decrypt_coeffs(g.import_(arr, level, 1.0)), np.array([float(x) for x in w]))
    if level == 2:
        bad = I.residues(3, (2, level + 1, g.n), g.moduli[: level + 1])
        for f in (g.decrypt, g.decrypt_coeffs):
            with pytest.raises(he.HEError) as e:
                f(g.import_(bad, level, 1.0))
            assert e.value.name == "HE_ESCALE"
    g.close()


@pytest.mark.parametrize("log_n", [12, 15])
def test_export_of_every_size_and_alignment(log_n):
    """64 KiB to 6.5 MB through the pinned slots: every level is the prefix of the whole, into buffers at
    any 8-byte offset, and nothing beside the buffer is written"""
    import ctypes
    import torch
    assert torch.cuda.is_available()
    from paper_2207_04620_amd import he
    ctx = he.Context(I.small(log_n=log_n, n_q=13, alpha=4, q_bits=45, p_bits=60))
    ct = ctx.encrypt(np.linspace(-1, 1, 64), nonce=5)
    whole = ctx.export(ct)
    back = ctx.import_(whole, ct.level, ct.scale)
    assert np.array_equal(ctx.decrypt(back, 64), ctx.decrypt(ct, 64))
    for level in range(13):
        low = ctx.drop(ct, level)
        size = 2 * (level + 1) << log_n
        for offset in (1, 255, 512):
            buf = np.full(offset + size + 3, 7, np.uint64)
            out = buf[offset:offset + size]
            assert he.lib().he_ct_export(ctx.ptr, low.ptr, out.ctypes.data_as(ctypes.POINTER(ctypes.c_uint64)), size) == 0
            assert np.array_equal(out.reshape(2, level + 1, -1), whole[:, :level + 1])
            assert (buf[:offset] == 7).all() and (buf[offset + size:] == 7).all()
    ctx.close()
