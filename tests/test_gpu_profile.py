"""The event profiler brackets every kernel launch: the launches it counts for one call are the call's kernels, in the
whole-row rings, the two-pass rings in either arithmetic and a ring of plain steps.
"""
import pytest

from gpu_common import to_dev
from test_gpu_ring14_rules import launches
from test_gpu_ring_block import Env
from workloads import gaussian_error, ternary_secret, uniform_residues

pytestmark = pytest.mark.gpu


# kernels of (encrypt, decrypt, rescale, mul_plain, keygen of one digit): whole rows; two passes with the row's
# element-wise work fused, in the fp64 and the integer arithmetic; two passes and separate element-wise kernels (an
# encryption expands s and e, transforms both in two launches and combines).  A key is two expansions and transforms, an
# automorphism and a combination.
@pytest.mark.parametrize("log_n,bits,want", [(12, 50, (1, 1, 2, 1, 6)), (13, 50, (1, 1, 2, 1, 6)),
                                             (14, 50, (2, 2, 4, 1, 8)), (16, 50, (2, 2, 4, 1, 8)),
                                             (12, 59, (2, 2, 4, 1, 8)), (16, 59, (2, 2, 4, 1, 8)),
                                             (11, 50, (5, 5, 7, 1, 8))])
def test_launches_are_all_counted(log_n, bits, want):
    env = Env((log_n, 3, 1, 1, bits))
    ctx, L = env.ctx, 3
    s, e = to_dev(ternary_secret(env.g, env.n)), to_dev(gaussian_error(env.g, env.n))
    a = to_dev(uniform_residues(env.g, ctx.q[:L], env.n))
    ka = to_dev(uniform_residues(env.g, ctx.primes, env.n, lead=(1,)))
    ke = to_dev(gaussian_error(env.g, (1, env.n)))
    ct, pt = env.buf(env.ct(L)), env.buf(env.ct(L)[:1])
    calls = [lambda: ctx.encrypt(s, pt, a, e), lambda: ctx.decrypt(s, ct), lambda: ctx.rescale(ct),
             lambda: ctx.mul_plain(ct, pt), lambda: ctx.keygen_galois(s, 5, ka, ke)]
    assert tuple(sum(launches(ctx, f).values()) for f in calls) == want
