"""N = 2^14, the ring on the border between the whole-row and the two-pass kernels: each step bit for bit against the
oracle on both sides of its rule, with the side it took read from the event profiler (a whole-row step has no column
passes of its own).  Ciphertexts and keys are uniform residues.
"""
import dataclasses

import numpy as np
import pytest

import test_gpu_attention as attention
from gpu_common import to_dev, to_host
from test_gpu_ring_block import Env
from workloads import rng, uniform_residues

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return Env((14, 12, 4, 3, 50))


def launches(ctx, fn):
    ctx.profile(True)
    ctx.profile_reset()
    fn()
    seen = {k: v[1] for k, v in ctx.profile_all().items()}
    ctx.profile(False)
    return seen


@pytest.mark.parametrize("limbs,count", [(12, 1), (1, 2), (9, 9), (12, 27)])
def test_key_switching_takes_two_passes(env, limbs, count):
    # (9, 9) and (12, 27): the short batches and the long ones
    c, key = env.ct(limbs), env.key()
    dev, steps = to_dev(key), [1 + 5 * r for r in range(count)]
    outs = env.ctx.rotate_hoisted(env.buf(c), steps, [dev] * count)
    for r in sorted({0, count - 1}):
        assert np.array_equal(to_host(outs[r].data), env.ck.rotate(c, steps[r], key)), r
    seen = launches(env.ctx, lambda: env.ctx.rotate_hoisted(env.buf(c), steps, [dev] * count))
    assert seen["ntt_inv_col"] == 2, seen     # the ModUp's and the ModDown's


@pytest.mark.parametrize("n_out,whole_rows", [(1, False), (2, False), (3, True), (5, True)])
def test_lazy_moddown(env, n_out, whole_rows):
    # 2 n_out polynomials of 12 limbs: 24, 48, 72 and 120 rows
    D, n1 = 16, 4
    T = env.n // 2 // D
    env.ctx.set_lazy_moddown(True)
    W = rng(71, 1).normal(0, 0.02, (D, n_out * D))
    keys = {s: env.key() for s in [T * b for b in range(1, n1)] + [T * n1 * g for g in range(1, D // n1)]}
    dev = {s: to_dev(k) for s, k in keys.items()}
    c = env.ct(12)

    def run():
        return env.ctx.linear_project([env.buf(c)], to_dev(W), T, n1, dev)

    outs = run()
    want = env.ck.linear_project([c], W, T, n1, keys, out_blocks=[0, n_out - 1], lazy=True)
    for j, w in zip((0, n_out - 1), want):
        assert np.array_equal(to_host(outs[j].data), w), j
    seen = launches(env.ctx, run)
    env.ctx.set_lazy_moddown(False)
    # inverse column passes: the baby steps' ModUp and ModDown, the giant steps' ModUp, the rescale's top limbs, and the
    # lazy ModDown's
    assert seen["ntt_inv_col"] == (4 if whole_rows else 5), seen


def test_moddown_of_one_polynomial(env):
    x = uniform_residues(env.g, env.ctx.q + env.ctx.p, env.n)
    dx = to_dev(x)
    assert np.array_equal(to_host(env.ctx.moddown(dx, 11)), env.ck.moddown(x, 11))
    assert launches(env.ctx, lambda: env.ctx.moddown(dx, 11))["ntt_inv_col"] == 1


@pytest.mark.parametrize("polys,limbs", [(16, 8), (43, 3)])   # 128 rows in two passes, 129 whole
def test_transforms(env, polys, limbs):
    x = uniform_residues(env.g, env.ctx.q[:limbs], env.n, lead=(polys,))
    t = env.ctx.ntt(to_dev(x))
    for b in (0, polys - 1):
        assert np.array_equal(to_host(t)[b], env.ck.ntt(x[b], list(range(limbs)))), b
    seen = launches(env.ctx, lambda: env.ctx.intt(t))
    assert np.array_equal(to_host(t), x)
    assert ("ntt_inv_col" in seen) == (polys * limbs <= 128), seen


def test_rescales_of_many_ciphertexts():
    # the weighted sums rescale 32 and 31 ciphertexts of six limbs at once (320 and 310 rows: whole rows); a single
    # rescale never has 128.  The noise in the slots grows at most with N: twice the bounds of N = 2^13.
    cfg = dataclasses.replace(attention.ATTN_TOY, name="attn14", log_n=14, tokens=32, head_dim=32)
    es, eo = attention.run_parity(cfg, 1, 1, [0])
    assert es <= 2.0 ** -28 and eo <= 2.0 ** -25
