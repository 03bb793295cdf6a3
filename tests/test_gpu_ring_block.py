"""The whole-row kernels of the rings N = 2^12 .. 2^14 bit for bit against the oracle, at the sizes where they can go
wrong: each ring, short last digits, more source limbs than one sum of eight terms takes (9 special primes, a digit
of 10), the same calls at N = 2^14, where transforms of many rows take them and the other steps the two-pass kernels,
more blocks than the CUs, and an output that is an input's buffer.
Ciphertexts and keys are uniform residues, which is all these steps see of them.
"""
import ctypes

import numpy as np
import pytest

from gpu_common import require_gpu, to_dev, to_host
from oracle import Ckks
from workloads import gaussian_error, rng, ternary_secret, uniform_residues

pytestmark = pytest.mark.gpu

# (log_n, n_q, n_p, dnum, bits)
CHAINS = [(12, 5, 2, 3, 50), (12, 10, 9, 1, 50), (13, 6, 2, 3, 50), (13, 5, 3, 2, 36), (14, 12, 4, 3, 50),
          (14, 3, 1, 3, 45)]


class Env:
    def __init__(self, chain):
        require_gpu()
        from paper_2609_12378_amd import Buf, Context
        log_n, n_q, n_p, dnum, bits = chain
        self.Buf = Buf
        self.ctx = Context(log_n, n_q, n_p, dnum, q_bits=bits)
        self.ck = Ckks(log_n, self.ctx.q, self.ctx.p, dnum)
        self.g = rng(40 + log_n, 1, extra=n_q)
        self.dnum, self.n_q, self.n = dnum, n_q, 1 << log_n

    def ct(self, limbs):
        return uniform_residues(self.g, self.ctx.q[:limbs], self.n, lead=(2,))

    def key(self):
        return uniform_residues(self.g, self.ctx.primes, self.n, lead=(self.dnum, 2))

    def buf(self, x):
        return self.Buf(to_dev(x), 1.0)


@pytest.fixture(scope="module", params=CHAINS, ids=lambda c: "n%d_%d+%d_dnum%d" % c[:4])
def env(request):
    return Env(request.param)


@pytest.mark.parametrize("rows", [1, 3, 64])
def test_transforms(env, rows):
    limbs = min(env.n_q, 5)                      # 64 x 5 rows: past the 128 of N = 2^14
    idx = list(range(limbs))
    x = uniform_residues(env.g, env.ctx.q[:limbs], env.n, lead=(rows,))
    t = env.ctx.ntt(to_dev(x))
    got = to_host(t)
    for b in sorted({0, rows - 1}):
        assert np.array_equal(got[b], env.ck.ntt(x[b], idx)), b
    back = to_host(env.ctx.intt(t))
    assert np.array_equal(back, x)


def test_hoisted_rotations(env):
    levels = sorted({env.n_q, max(1, env.n_q - 2), 1})
    keys = [env.key() for _ in range(3)]
    dev = [to_dev(k) for k in keys]
    for limbs in levels:
        for count in (1, 3, 32):
            c = env.ct(limbs)
            steps = [1 + 5 * r for r in range(count)]
            outs = env.ctx.rotate_hoisted(env.buf(c), steps, [dev[r % 3] for r in range(count)])
            for r in sorted({0, count // 2, count - 1}):
                assert np.array_equal(to_host(outs[r].data), env.ck.rotate(c, steps[r], keys[r % 3])), (limbs, count, r)


def test_mul_relin_rescale(env):
    limbs = env.n_q
    a, b, rlk = env.ct(limbs), env.ct(limbs), env.key()
    want = env.ck.mul_relin(a, b, rlk)
    da, db, dk = env.buf(a), env.buf(b), to_dev(rlk)
    out = env.ctx.mul_relin(da, db, dk)
    assert np.array_equal(to_host(out.data), want)
    if limbs > 1:
        assert np.array_equal(to_host(env.ctx.rescale(out).data), env.ck.rescale(want))
    # the output over the first input
    ca, cb = da.c(env.n), db.c(env.n)
    assert env.ctx.lib.ckks_mul_relin(env.ctx.h, ctypes.byref(ca), ctypes.byref(cb), ctypes.c_void_p(dk.data_ptr()),
                                      ctypes.byref(ca)) == 0
    assert np.array_equal(to_host(da.data), want)


def test_modup_moddown(env):
    import torch
    level = env.n_q - 1
    L, ext = level + 1, level + 1 + env.ctx.n_p
    c = env.ct(L)[0]
    want = env.ck.modup(c, level)
    assert np.array_equal(to_host(env.ctx.modup(to_dev(c), level)), want)
    # the polynomial inside the buffer that takes its digits
    d = torch.zeros(want.shape, dtype=torch.uint64, device="cuda")
    d.view(torch.int64).reshape(-1, env.n)[:L] = to_dev(c).view(torch.int64)
    p = ctypes.c_void_p(d.data_ptr())
    assert env.ctx.lib.ckks_modup(env.ctx.h, p, level, p) == 0
    assert np.array_equal(to_host(d), want)
    x = uniform_residues(env.g, env.ctx.q[:L] + env.ctx.p, env.n)
    assert x.shape[0] == ext
    assert np.array_equal(to_host(env.ctx.moddown(to_dev(x), level)), env.ck.moddown(x, level))


def test_encrypt_decrypt(env):
    s = ternary_secret(env.g, env.n)
    for limbs in sorted({1, env.n_q}):
        m = env.ct(limbs)[:1]
        a = uniform_residues(env.g, env.ctx.q[:limbs], env.n)
        e = gaussian_error(env.g, env.n)
        want = env.ck.encrypt(s, m[0], a, e)
        ct = env.ctx.encrypt(to_dev(s), env.buf(m), to_dev(a), to_dev(e))
        assert np.array_equal(to_host(ct.data), want)
        assert np.array_equal(to_host(env.ctx.decrypt(to_dev(s), ct).data[0]), env.ck.decrypt(s, want))


def test_encode_with_large_coefficients(env):
    # a few coefficients beyond 2^52: the general reduction of the waves that hold them
    z = env.g.uniform(-1, 1, env.n // 2)
    limbs = min(env.n_q, 3)
    scale = 2.0 ** 57
    pt = env.ctx.encode(to_dev(z), None, scale, limbs)
    assert np.array_equal(to_host(pt.data[0]), env.ck.encode(z, None, scale, limbs))
