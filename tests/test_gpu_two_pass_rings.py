"""The two-pass rings N = 2^15 and 2^16 bit for bit against the oracle where the fused passes can go wrong: digits of
more than eight limbs, short last digits, 59-bit (integer) moduli, a chain whose top prime needs the integer arithmetic
and the others do not, and both sides of the rule that splits the largest batches of rotations off (27 and 28 rotations
of seven limbs at N = 2^16).  Then the one-vector FFT of every ring size, and the projections that run several giant steps a
launch.  Ciphertexts and keys are uniform residues.
"""
import dataclasses

import numpy as np
import pytest

import test_gpu_project as fm
import test_gpu_project_tm as tm
from gpu_common import require_gpu, to_dev, to_host
from oracle import Ckks
from oracle.ckks import gen_primes
from test_gpu_ring_block import Env
from workloads import TOY, gaussian_error, rng, ternary_secret, uniform_residues

pytestmark = pytest.mark.gpu


class MixedEnv(Env):
    """Fp64 primes below one 59-bit top prime: a rescale's source and targets take different arithmetics."""

    def __init__(self, log_n):
        require_gpu()
        from paper_2609_12378_amd import Buf, Context
        small, big = gen_primes(45, 2 << log_n, 4), gen_primes(59, 2 << log_n, 3)
        self.Buf = Buf
        self.ctx = Context(log_n, 4, 2, 2, q=list(small[:3]) + [big[0]], p=list(big[1:3]))
        self.ck = Ckks(log_n, self.ctx.q, self.ctx.p, 2)
        self.g = rng(40 + log_n, 1, extra=77)
        self.dnum, self.n_q, self.n = 2, 4, 1 << log_n


# (log_n, n_q, n_p, dnum, bits), or a mixed chain's log_n
CHAINS = [(15, 5, 2, 3, 50), (15, 10, 10, 1, 50), (15, 4, 2, 2, 59), (16, 5, 2, 3, 50), (16, 10, 10, 1, 50),
          (16, 4, 2, 2, 59), 12, 15]


@pytest.fixture(scope="module", params=CHAINS, ids=str)
def env(request):
    return MixedEnv(request.param) if isinstance(request.param, int) else Env(request.param)


def test_rotations(env):
    keys = [env.key() for _ in range(2)]
    dev = [to_dev(k) for k in keys]
    for limbs in sorted({env.n_q, 1}):
        for count in (1, 4, 5):
            c = env.ct(limbs)
            steps = [1 + 3 * r for r in range(count)]
            outs = env.ctx.rotate_hoisted(env.buf(c), steps, [dev[r % 2] for r in range(count)])
            for r in sorted({0, count - 1}):
                assert np.array_equal(to_host(outs[r].data), env.ck.rotate(c, steps[r], keys[r % 2])), (limbs, count, r)


def test_finishing_kernels_of_large_batches():
    # waves: 896 a rotation, the line at 24576
    env = Env((16, 7, 3, 3, 50))
    c, key = env.ct(7), env.key()
    dev = to_dev(key)
    for count in (27, 28):
        steps = [1 + 3 * r for r in range(count)]
        outs = env.ctx.rotate_hoisted(env.buf(c), steps, [dev] * count)
        for r in (0, count - 1):
            assert np.array_equal(to_host(outs[r].data), env.ck.rotate(c, steps[r], key)), (count, r)


def test_mul_relin_rescale_modup_moddown(env):
    a, b, rlk = env.ct(env.n_q), env.ct(env.n_q), env.key()
    want = env.ck.mul_relin(a, b, rlk)
    out = env.ctx.mul_relin(env.buf(a), env.buf(b), to_dev(rlk))
    assert np.array_equal(to_host(out.data), want)
    assert np.array_equal(to_host(env.ctx.rescale(out).data), env.ck.rescale(want))
    level = env.n_q - 2                       # a short last digit
    c = env.ct(level + 1)[0]
    assert np.array_equal(to_host(env.ctx.modup(to_dev(c), level)), env.ck.modup(c, level))
    x = uniform_residues(env.g, env.ctx.q[:level + 1] + env.ctx.p, env.n)
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


@pytest.mark.parametrize("log_n", [11, 12, 13, 14, 15, 16])
@pytest.mark.parametrize("bits", [50, 59])
def test_one_vector_fft(log_n, bits):
    """Encoded integers equal the oracle's; decoded slots agree with the oracle's decode of the same integers and return
    the input.  A radix-2 transform of M = N/2 points adds at most 5 u relative to the 2-norm a stage, which |z| <= sqrt(2)
    bounds by sqrt(2 M): that twice between two decodes (4.5e-12 at N = 2^16), and between the input and its decode, where
    the rounding of N coefficients adds at most N/2 over the scale (9.3e-10)."""
    require_gpu()
    from paper_2609_12378_amd import Context
    ctx = Context(log_n, 3, 1, 3, q_bits=bits)
    ck = Ckks(log_n, ctx.q, ctx.p, 3)
    M, scale = ctx.n // 2, 2.0 ** 45
    g = rng(60 + log_n, 1)
    z = g.uniform(-1, 1, (2, M))
    fp = 2 * 5 * log_n * 2.0 ** -53 * np.sqrt(2 * M)
    trip = fp + ctx.n / 2 / scale
    for im in (None, z[1]):
        for limbs in (1, 2, 3):
            pt = ctx.encode(to_dev(z[0]), None if im is None else to_dev(im), scale, limbs)
            want = ck.encode(z[0], im, scale, limbs)
            assert np.array_equal(to_host(pt.data[0]), want), (limbs, im is None)
            re_, im_ = (to_host(v) for v in ctx.decode(pt))
            assert np.max(np.abs(re_ - z[0])) <= trip and np.max(np.abs(im_ - (0 if im is None else im))) <= trip
            zo = ck.decode(want, scale)
            assert np.max(np.abs(re_ - zo.real)) <= fp and np.max(np.abs(im_ - zo.imag)) <= fp


RING128 = dataclasses.replace(TOY, name="runs128", tokens=128)


@pytest.mark.parametrize("cfg,n_in,n_out,n1,lazy", [
    (TOY, 1, 11, 16, False),       # five giant steps a launch: 55 rows, the second row group short; then three
    (TOY, 1, 5, 16, True),         # all eight in one launch: 40 rows
    (TOY, 3, 2, 32, True),         # 192 kappa in chunks of 64, an odd number of steps; eight rows
    (RING128, 2, 3, 4, False),     # 16 features in runs of 128 positions: one polynomial per block
], ids=["55rows", "40rows_lazy", "chunks", "runs128"])
def test_token_major_giant_step_groups(cfg, n_in, n_out, n1, lazy):
    D = (1 << cfg.log_n) // 2 // cfg.tokens
    assert tm.run_case(cfg, n_in * D, n_out * D, n1, [0, n_out - 1], lazy=lazy) <= 2.0 ** -12


def test_token_major_weights_beyond_2_52(monkeypatch):
    # encoded coefficients beyond 2^52 (about 2^36 57/128 2^18): the exact reduction of the blocks that hold one; the
    # projection is linear in the weights, so the bound of the other cases scales with them
    plain = tm.gaussian_weights
    monkeypatch.setattr(tm, "gaussian_weights", lambda *a: plain(*a) * 2.0 ** 18)
    assert tm.run_case(TOY, TOY.feats, TOY.feats, 16, [0]) <= 2.0 ** (18 - 12)


@pytest.mark.parametrize("log_n", [15, 16])
def test_a_nan_weight_stays_in_its_plaintext(log_n):
    # its diagonal's transform is all NaN, which the integer conversion of a coefficient takes to zero: as if the diagonal
    # W[(o + 1) mod D][o] were zero, and canonical residues everywhere
    require_gpu()
    from paper_2609_12378_amd import Buf, Context
    D, n1, L = 4, 2, 2
    ctx = Context(log_n, 2, 1, 2, q_bits=50)
    T = ctx.n // 2 // D
    g = rng(61, 2)
    W = g.normal(0, 0.02, (D, D))
    Z = W.copy()
    Z[(np.arange(D) + 1) % D, np.arange(D)] = 0.0
    W[2, 1] = np.nan
    ct = Buf(to_dev(uniform_residues(g, ctx.q[:L], ctx.n, lead=(2,))), 2.0 ** 40)
    key = to_dev(uniform_residues(g, ctx.primes, ctx.n, lead=(2, 2)))
    out = [to_host(ctx.linear_project([ct], to_dev(M), T, n1, {T: key, 2 * T: key})[0].data) for M in (W, Z)]
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("lazy", [False, True])
@pytest.mark.parametrize("n1", [16, 24])
def test_feature_major_giant_step_groups(n1, lazy):
    # n1 = 16: several giant steps a launch; 24 does not divide D, so the last one stands alone
    cfg = dataclasses.replace(TOY, n1=n1)
    assert fm.run_case(cfg, TOY.feats, 2 * TOY.feats, [0, 1], lazy=lazy) <= 2.0 ** -12


def test_token_major_smaller_workspace():
    """A workspace without room for eight giant steps a launch takes fewer; one without room for any is refused."""
    require_gpu()
    import torch
    from paper_2609_12378_amd import Buf, CkksError, Context
    cfg, n1 = TOY, 16
    ctx = Context(cfg.log_n, cfg.n_q, cfg.n_p, cfg.dnum, q_bits=cfg.q_bits)
    n, T, L, D = ctx.n, cfg.tokens, cfg.level + 1, cfg.feats
    g = rng(60, 2)
    ct = Buf(to_dev(uniform_residues(g, ctx.q[:L], n, lead=(2,))), 2.0 ** 30)
    W = to_dev(g.normal(0, 0.02, (D, D)))
    key = to_dev(uniform_residues(g, ctx.primes, n, lead=(cfg.dnum, 2)))
    keys = {s: key for s in [*range(1, n1), *range(-D, n1 - D), *range(n1, D, n1)]}
    want = to_host(ctx.linear_project([ct], W, T, n1, keys, layout="tm")[0].data)
    need = ctx.workspace_bytes(ctx.OP_LINEAR_PROJECT_TM, (L, T, D, D, n1))
    # four rows' accumulators and rotations less: room for four giant steps
    ctx.set_workspace(torch.empty(need // 8 - 2 * 4 * 2 * L * n, dtype=torch.uint64, device="cuda"))
    assert np.array_equal(to_host(ctx.linear_project([ct], W, T, n1, keys, layout="tm")[0].data), want)
    ctx.set_workspace(torch.empty(4096, dtype=torch.uint64, device="cuda"))
    with pytest.raises(CkksError, match="too small"):
        ctx.linear_project([ct], W, T, n1, keys, layout="tm")
    ctx.set_workspace(None)
