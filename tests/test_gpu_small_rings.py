"""Key switching and the projections in the rings below N = 2^12 bit for bit against the oracle, in the fp64, the forced
integer and the 59-bit arithmetic.  N = 2^8 is one row of 256 points without a column pass, so the kernels that finish
a two-pass transform's row do not apply to it; 2^4 is the smallest ring, 2^9 and 2^11 have rows of 32 and 128 points.
Ciphertexts and keys are uniform residues.
"""
import pytest

import numpy as np
from gpu_common import to_dev, to_host
from test_gpu_ring_block import Env
from workloads import rng, uniform_residues

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[(n, a) for n in (4, 8, 9, 11) for a in ("fp64", "integer", "59bit")],
                ids=lambda p: "n%d_%s" % p)
def env(request):
    log_n, arith = request.param
    e = Env((log_n, 4, 2, 2, 59 if arith == "59bit" else 50))
    e.ctx.set_ntt_arith(1 if arith == "integer" else 0)
    e.fp64 = arith == "fp64"
    return e


def test_mul_relin(env):
    for limbs in (4, 3, 1):                   # two full digits, a short one, a single limb
        a, b, rlk = env.ct(limbs), env.ct(limbs), env.key()
        out = env.ctx.mul_relin(env.buf(a), env.buf(b), to_dev(rlk))
        assert np.array_equal(to_host(out.data), env.ck.mul_relin(a, b, rlk)), limbs


def test_rotations(env):
    keys = [env.key() for _ in range(2)]
    dev = [to_dev(k) for k in keys]
    kb = uniform_residues(env.g, env.ctx.primes, env.n, lead=(env.dnum,))
    seeds = [(5, 9), (1, 2 ** 63)]
    for limbs in (4, 3):
        c, steps = env.ct(limbs), [1, -2]
        for r, o in enumerate(env.ctx.rotate_hoisted(env.buf(c), steps, dev)):
            assert np.array_equal(to_host(o.data), env.ck.rotate(c, steps[r], keys[r])), (limbs, r)
        out = env.buf(np.zeros_like(c))
        env.ctx.rotate_noalloc(env.buf(c), 3, dev[0], out)
        assert np.array_equal(to_host(out.data), env.ck.rotate(c, 3, keys[0])), limbs
        for r, o in enumerate(env.ctx.rotate_hoisted_seeded(env.buf(c), steps, [to_dev(kb)] * 2, seeds)):
            want = env.ck.rotate(c, steps[r], env.ck.seeded_key(kb, seeds[r]))
            assert np.array_equal(to_host(o.data), want), (limbs, r)


@pytest.mark.parametrize("lazy", [False, True])
def test_projections(env, lazy):
    slots = env.n // 2
    D = min(16, slots // 2)
    T, n1 = slots // D, max(2, D // 4)
    n2 = D // n1
    env.ctx.set_lazy_moddown(lazy)
    W = rng(70, 1).normal(0, 0.02, (D, 2 * D))
    for layout in ("fm", "tm") if env.fp64 and env.n >= 256 else ("fm",):   # the library's own limits
        if layout == "fm":
            steps = [T * b for b in range(1, n1)] + [T * n1 * g for g in range(1, n2)]
        else:
            steps = [*range(1, n1), *range(-D, n1 - D), *range(n1, D, n1)]
        keys = {s: env.key() for s in steps}
        c = env.ct(3)
        want = getattr(env.ck, "linear_project" if layout == "fm" else "linear_project_tm")(
            [c], W, T, n1, keys, out_blocks=[0, 1], lazy=lazy)
        outs = env.ctx.linear_project([env.buf(c)], to_dev(W), T, n1, {s: to_dev(k) for s, k in keys.items()},
                                      layout=layout)
        for o, w in zip(outs, want):
            assert np.array_equal(to_host(o.data), w), layout
    env.ctx.set_lazy_moddown(False)
