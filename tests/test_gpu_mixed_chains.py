"""Rotations in fp64 chains whose primes differ in size, bit for bit against the oracle: a conversion from a source of
twice a target or more, or from more than 16 sources, is not done in fp64, and each step of a key switch takes the fused
kernels that its own primes and conversion allow.  The launches of one rotation, read from the event profiler, show
which were taken.  Ciphertexts and keys are uniform residues.
"""
import numpy as np
import pytest

from gpu_common import require_gpu, to_dev, to_host
from oracle import Ckks
from oracle.ckks import gen_primes
from test_gpu_ring_block import Env
from workloads import rng, uniform_residues

pytestmark = pytest.mark.gpu


def chain(log_n, kind):
    """(q, p, dnum, digits, the ModDown's conversion is fp64)"""
    b50, b40 = gen_primes(50, 2 << log_n, 40), gen_primes(40, 2 << log_n, 8)
    if kind == "special50":          # special primes of 50 bits over scale primes of 40: the ModDown is not fp64
        return [b50[0], *b40[:3]], b50[1:3], 2, 2, False
    if kind == "base50":             # only the first digit's conversion is not
        return [b50[0], *b40[:3]], b40[3:5], 2, 2, True
    return b50[:17], b50[17:34], 1, 1, False    # 17 sources


class Chain(Env):
    def __init__(self, log_n, kind):
        require_gpu()
        from paper_2609_12378_amd import Buf, Context
        q, p, dnum, self.digits, self.down_f64 = chain(log_n, kind)
        self.Buf = Buf
        self.ctx = Context(log_n, len(q), len(p), dnum, q=[int(x) for x in q], p=[int(x) for x in p])
        self.ck = Ckks(log_n, self.ctx.q, self.ctx.p, dnum)
        self.g = rng(80 + log_n, 1, extra=len(q))
        self.dnum, self.n_q, self.n = dnum, len(q), 1 << log_n


@pytest.mark.parametrize("log_n", [12, 15, 16])
@pytest.mark.parametrize("kind", ["special50", "base50", "sources17"])
def test_rotations(log_n, kind):
    env = Chain(log_n, kind)
    keys = [env.key() for _ in range(2)]
    dev = [to_dev(k) for k in keys]
    kb, seed = uniform_residues(env.g, env.ctx.primes, env.n, lead=(env.dnum,)), (3, 4)
    for limbs, count in ((env.n_q, 5), (2, 1)):
        c = env.ct(limbs)
        steps = [1 + 3 * r for r in range(count)]
        outs = env.ctx.rotate_hoisted(env.buf(c), steps, [dev[r % 2] for r in range(count)])
        for r in sorted({0, count - 1}):
            assert np.array_equal(to_host(outs[r].data), env.ck.rotate(c, steps[r], keys[r % 2])), (limbs, r)
        out = env.ctx.rotate_hoisted_seeded(env.buf(c), steps[:1], [to_dev(kb)], [seed])[0]
        assert np.array_equal(to_host(out.data), env.ck.rotate(c, steps[0], env.ck.seeded_key(kb, seed))), limbs

    # one rotation: the inverse row passes are the ModUp's digits' alone, the P rows' ones run in their inner products;
    # the converted rows' column pass is a launch of its own only where the conversion is (2^12: whole-row transforms)
    if log_n == 12:
        return
    c = env.buf(env.ct(env.n_q))
    env.ctx.profile(True)
    env.ctx.profile_reset()
    env.ctx.rotate(c, 1, dev[0])
    seen = {k: v[1] for k, v in env.ctx.profile_all().items()}
    env.ctx.profile(False)
    assert seen["ntt_inv_row"] == env.digits and seen["ntt_inv_col"] == env.digits + 1, seen
    fused = log_n == 16 and env.down_f64
    assert seen["ntt_fwd_col"] == (1 if fused else 2), seen
