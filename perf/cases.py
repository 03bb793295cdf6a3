"""The calls a program makes of this library, as cases that can be timed and compared.

Every case goes through the public binding (``Context``).  Seven kinds of use:

* ``client``   one slot vector there and back: encode, encrypt, decrypt, decode;
* ``ops``      one evaluation step on ciphertexts: multiply and relinearise, rescale, rotate, add, multiply by a
               plaintext, rescale (a polynomial activation or a masked rotate-and-add);
* ``hoist``    rotations of one ciphertext that share a ModUp;
* ``ntt``      batched transforms, one buffer forward and another backward;
* ``fm``/``tm``  the packed projection in the feature-major and in the token-major layout;
* ``attn``     one key/value head's scores and the weighted sums that consume them.

A context is the handle a program keeps, so states with the same parameters share one.  Residues (ciphertexts, keys)
are uniform modulo their primes, as real ones are; slots are uniform on [-1, 1], weights N(0, 0.02^2), secrets
ternary and errors rounded N(0, 3.2^2).
"""
import functools
import math

import numpy as np
import torch

from paper_2609_12378_amd import Buf, Context


def listed():
    return [
        # the smallest call a client makes: one vector of the toy ring (2^12, four 36-bit primes); launches count
        dict(name="client_n12", kind="client", log_n=12, limbs=4, bits=36, scale_log2=30, imag=False),
        # the client of the projection: a level-12 input of the large ring, complex slots
        dict(name="client_n16", kind="client", log_n=16, limbs=13, bits=50, scale_log2=40, imag=True),
        # one evaluation step in a small ring (the small attention ring's chain)
        dict(name="ops_n13", kind="ops", log_n=13, n_q=6, n_p=2, dnum=3, bits=50, limbs=6),
        # the same step at the projection's ring and level
        dict(name="ops_n16", kind="ops", log_n=16, n_q=24, n_p=8, dnum=3, bits=50, limbs=13),
        # the key-switching benchmark: 32 hoisted rotations at the top level into buffers the program keeps
        dict(name="hoist32_n16", kind="hoist", log_n=16, n_q=24, n_p=8, dnum=3, bits=50, limbs=24, count=32,
             keep=True),
        # a few rotations in a medium ring at a level that leaves the last digit short, outputs from the call
        dict(name="hoist9_n14", kind="hoist", log_n=14, n_q=11, n_p=4, dnum=3, bits=50, limbs=9, count=9, keep=False),
        # the paper's prime sizes (59-bit chain, 60-bit special primes, dnum 5) at its top level
        dict(name="hoist8_paper", kind="hoist", log_n=16, n_q=37, n_p=8, dnum=5, bits=59, limbs=37, count=8,
             keep=False),
        # the transform benchmark's batch, both directions
        dict(name="ntt_n16", kind="ntt", log_n=16, limbs=36, bits=50, batch=64),
        # an attention-output projection (4096 x 4096) in the feature-major layout, 128 tokens, level 12
        dict(name="fm_n16", kind="fm", log_n=16, n_q=24, n_p=8, dnum=3, bits=50, limbs=13, feats=256, n_in=16,
             n_out=16, n1=32, lazy=True),
        # a projection in a medium ring: 1024 x 768, 32 tokens
        dict(name="fm_n14", kind="fm", log_n=14, n_q=7, n_p=3, dnum=3, bits=50, limbs=7, feats=256, n_in=4, n_out=3,
             n1=16, lazy=False),
        # the attention-output projection in the token-major layout
        dict(name="tm_n16", kind="tm", log_n=16, n_q=24, n_p=8, dnum=3, bits=50, limbs=13, feats=256, n_in=16,
             n_out=16, n1=16, lazy=True),
        # one key/value head with the two query ciphertexts that share it: scores, then the weighted sums
        dict(name="attn_n16", kind="attn", log_n=16, n_q=24, n_p=8, dnum=3, bits=50, limbs=13, tokens=128,
             head_dim=128, queries=2),
    ]


def _spread(rng, lo, hi):
    """An integer of [lo, hi], evenly over the logarithm."""
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def _chain(rng, least, most, bits):
    """A prime chain with its digits: as many special primes as the largest digit has limbs (at most 8)."""
    n_q = rng.randint(least, most)
    dnum = rng.randint(max(1, -(-n_q // 8)), min(5, n_q))
    return dict(n_q=n_q, n_p=min(8, -(-n_q // dnum)), dnum=dnum, bits=bits)


def draw(rng):
    kind = rng.choice(["client", "client", "ops", "ops", "ops", "hoist", "hoist", "hoist", "ntt", "ntt", "fm", "tm",
                       "attn"])
    log_n = rng.randint(12, 16)
    bits = rng.choice([36, 45, 50, 50, 59])
    if kind == "client":
        return dict(kind=kind, log_n=log_n, limbs=rng.randint(1, 24), bits=bits, scale_log2=30 if bits < 40 else 40,
                    imag=rng.random() < 0.5)
    if kind == "ops":
        c = dict(kind=kind, log_n=log_n, **_chain(rng, 3, 24, bits))
        return dict(c, limbs=rng.randint(3, c["n_q"]))
    if kind == "hoist":
        c = dict(kind=kind, log_n=log_n, **_chain(rng, 3, 37, bits))
        return dict(c, limbs=rng.randint(1, c["n_q"]), count=_spread(rng, 1, 32), keep=rng.random() < 0.5)
    if kind == "ntt":
        return dict(kind=kind, log_n=log_n, limbs=_spread(rng, 1, 36), bits=bits, batch=_spread(rng, 1, 64))
    # projections and attention in the rings below the largest
    log_n = rng.randint(12, 15)
    if kind in ("fm", "tm"):
        bits = bits if kind == "fm" else min(bits, 50)
        c = dict(kind=kind, log_n=log_n, **_chain(rng, 3, 13, bits))
        return dict(c, limbs=rng.randint(2, c["n_q"]), feats=rng.choice([64, 128, 256]), n_in=rng.randint(1, 5),
                    n_out=rng.randint(1, 5), n1=rng.choice([8, 12, 16, 32]), lazy=rng.random() < 0.5)
    slots = 1 << (log_n - 1)
    tokens = rng.choice([t for t in (16, 32, 64) if t <= slots // t <= 256])
    feats = slots // tokens
    head = rng.choice([h for h in (16, 32, 64, 128) if tokens <= h <= feats])
    c = dict(kind=kind, log_n=log_n, **_chain(rng, 4, 8, min(bits, 50)))
    return dict(c, limbs=rng.randint(4, c["n_q"]), tokens=tokens, head_dim=head, queries=rng.randint(1, 3))


# ---- states -----------------------------------------------------------------------------------------------------

@functools.lru_cache(maxsize=4)
def _context(log_n, n_q, n_p, dnum, bits, lazy):
    # 59-bit chains take special primes of 60 bits; the others special primes of the same size
    ctx = Context(log_n, n_q, n_p, dnum, q_bits=bits, p_bits=60 if bits == 59 else bits)
    ctx.set_lazy_moddown(lazy)
    return ctx


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _residues(g, primes, n, *lead):
    q = torch.tensor(list(primes), dtype=torch.int64, device="cuda")
    x = torch.randint(0, 1 << 62, (*lead, len(primes), n), dtype=torch.int64, device="cuda", generator=g)
    return x.remainder_(q[:, None]).view(torch.uint64)


def _error(g, n):
    e = torch.randn(n, dtype=torch.float64, device="cuda", generator=g) * 3.2
    return e.round().clamp_(-19, 19).to(torch.int32)


def _key(g, ctx):
    return _residues(g, ctx.primes, ctx.n, ctx.dnum, 2)


def _ct(g, ctx, limbs, scale):
    return Buf(_residues(g, ctx.q[:limbs], ctx.n, 2), scale)


def _client_inputs(case, seed):
    """Slots, secret and error of a client case: what it draws before any prime is known."""
    g, n = _gen(seed), 1 << case["log_n"]
    z = torch.rand((2, n // 2), dtype=torch.float64, device="cuda", generator=g) * 2 - 1
    s = torch.randint(-1, 2, (n,), dtype=torch.int8, device="cuda", generator=g)
    return g, z[0].contiguous(), z[1].contiguous() if case["imag"] else None, s, _error(g, n)


def _project_steps(case):
    feats, n1 = case["feats"], case["n1"]
    tokens = (1 << (case["log_n"] - 1)) // feats
    n2 = -(-feats // n1)
    if case["kind"] == "fm":
        return tokens, [tokens * b for b in range(1, n1)] + [tokens * n1 * k for k in range(1, n2)]
    return tokens, [b for b in range(1, n1)] + [b - feats for b in range(n1)] + [n1 * k for k in range(1, n2)]


def prepare(case, seed):
    kind, n = case["kind"], 1 << case["log_n"]
    lazy = kind == "attn" or bool(case.get("lazy"))
    ctx = _context(case["log_n"], case.get("n_q", case["limbs"]), case.get("n_p", 0), case.get("dnum", 1),
                   case["bits"], lazy)
    st = {"kind": kind, "ctx": ctx}
    if kind == "client":
        g, re, im, s, e = _client_inputs(case, seed)
        return dict(st, re=re, im=im, s=s, e=e, a=_residues(g, ctx.q, n), scale=2.0 ** case["scale_log2"],
                    limbs=case["limbs"])
    g, limbs = _gen(seed), case["limbs"]
    if kind == "ops":
        pt = Buf(_residues(g, ctx.q[:limbs], n, 1), 2.0 ** 40)
        return dict(st, a=_ct(g, ctx, limbs, 2.0 ** 40), b=_ct(g, ctx, limbs, 2.0 ** 40), pt=pt, rlk=_key(g, ctx),
                    key=_key(g, ctx), step=5)
    if kind == "hoist":
        steps = list(range(1, case["count"] + 1))
        outs = None
        if case["keep"]:
            outs = [Buf(torch.empty((2, limbs, n), dtype=torch.uint64, device="cuda"), 1.0) for _ in steps]
        return dict(st, ct=_ct(g, ctx, limbs, 2.0 ** 40), steps=steps, keys=[_key(g, ctx) for _ in steps], outs=outs)
    if kind == "ntt":
        return dict(st, x=_residues(g, ctx.q, n, case["batch"]), y=_residues(g, ctx.q, n, case["batch"]))
    if kind in ("fm", "tm"):
        tokens, steps = _project_steps(case)
        d_in, d_out = case["n_in"] * case["feats"], case["n_out"] * case["feats"]
        W = torch.randn((d_in, d_out), dtype=torch.float64, device="cuda", generator=g) * 0.02
        return dict(st, cts=[_ct(g, ctx, limbs, 2.0 ** 40) for _ in range(case["n_in"])], W=W, tokens=tokens,
                    n1=case["n1"], keys={k: _key(g, ctx) for k in steps})
    steps = Context.attention_steps(n // 2, case["tokens"], case["head_dim"])
    return dict(st, q=[_ct(g, ctx, limbs, 2.0 ** 50) for _ in range(case["queries"])],
                k=[_ct(g, ctx, limbs, 2.0 ** 50)], v=[_ct(g, ctx, limbs, 2.0 ** 50)], tokens=case["tokens"],
                head_dim=case["head_dim"], rlk=_key(g, ctx), keys={k: _key(g, ctx) for k in steps})


def _res(b):
    """A buffer's residues as signed words (the same bits; every residue is below 2^63)."""
    return (b.data if isinstance(b, Buf) else b).view(torch.int64)


def run(st):
    ctx, kind = st["ctx"], st["kind"]
    if kind == "client":
        pt = ctx.encode(st["re"], st["im"], st["scale"], st["limbs"])
        ct = ctx.encrypt(st["s"], pt, st["a"], st["e"])
        back = ctx.decrypt(st["s"], ct)
        re, im = ctx.decode(back)
        return {"pt": _res(pt), "ct": _res(ct), "back": _res(back), "re": re, "im": im}
    if kind == "ops":
        x = ctx.rescale(ctx.mul_relin(st["a"], st["b"], st["rlk"]))
        y = ctx.rotate(x, st["step"], st["key"])
        z = ctx.rescale(ctx.mul_plain(ctx.add(x, y), st["pt"]))
        return [_res(x), _res(y), _res(z)]
    if kind == "hoist":
        return [_res(o) for o in ctx.rotate_hoisted(st["ct"], st["steps"], st["keys"], st["outs"])]
    if kind == "ntt":
        return [_res(ctx.ntt(st["x"])), _res(ctx.intt(st["y"]))]
    if kind in ("fm", "tm"):
        return [_res(o) for o in ctx.linear_project(st["cts"], st["W"], st["tokens"], st["n1"], st["keys"],
                                                    layout=kind)]
    of = [0] * len(st["q"])
    p = ctx.attention_scores(st["q"], st["k"], of, st["tokens"], st["head_dim"], st["rlk"], st["keys"])
    o = ctx.attention_apply(p, st["v"], of, st["tokens"], st["head_dim"], st["rlk"], st["keys"])
    return [_res(x) for x in p + o]


# ---- what a pass cannot do without ------------------------------------------------------------------------------

def _switch(case, limbs, rotations, modups=1):
    """(key bytes, modular products) of `rotations` key switches at `limbs` limbs that share `modups` ModUps."""
    n, log_n, K = 1 << case["log_n"], case["log_n"], case["n_p"]
    alpha = -(-case["n_q"] // case["dnum"])
    nd, ext = (limbs - 1) // alpha + 1, limbs + K
    half = n * log_n / 2                                   # butterflies of one row
    up = modups * (half * (limbs + nd * ext - limbs) + n * limbs * ext)
    down = 2 * (half * (K + limbs) + n * K * limbs + n * limbs)
    return 8.0 * rotations * nd * 2 * ext * n, up + rotations * (2.0 * nd * ext * n + down)


def work(case):
    """Bytes: each input and each output once.  flops: two for every modular product or FFT multiply-add."""
    kind, n, log_n, L = case["kind"], 1 << case["log_n"], case["log_n"], case["limbs"]
    half, row = n * log_n / 2, 8.0 * n
    if kind == "client":
        by = row * (2 if case["imag"] else 1.5) + n + 4 * n + row * (L + L + 2 * L + L)
        return {"bytes": by, "flops": 2 * (half * (L + 2 * L + L + min(L, 2)) + 4 * half + 4 * n * L)}
    if kind == "ops":
        k1, m1 = _switch(case, L, 1)
        k2, m2 = _switch(case, L - 1, 1)
        by = row * (4 * L + (L - 1) + 4 * (L - 1) + 2 * (L - 2)) + k1 + k2
        return {"bytes": by, "flops": 2 * (m1 + m2 + n * (4 * L + 2 * L) + 2 * half * 2 * L)}
    if kind == "hoist":
        k, m = _switch(case, L, case["count"])
        return {"bytes": row * 2 * L * (1 + case["count"]) + k, "flops": 2 * m}
    if kind == "ntt":
        rows = 2 * case["batch"] * L
        return {"bytes": 2 * row * rows, "flops": 2 * half * rows}
    if kind in ("fm", "tm"):
        D, n_in, n_out, n1 = case["feats"], case["n_in"], case["n_out"], case["n1"]
        n2 = -(-D // n1)
        baby = (n1 - 1) if kind == "fm" else 2 * n1 - 1
        kb, mb = _switch(case, L, baby)
        kg, mg = _switch(case, L, n2 - 1, n2 - 1)
        pts = n_in * n_out * D
        if kind == "fm":
            enc, mac = pts * (2 * half + half * L), pts * 2.0 * L * n
        else:
            enc, mac = 2 * pts * (D * math.log2(2 * D) * (1 + L)), pts * 4.0 * L * n
        by = row * (2 * L * n_in + 2 * (L - 1) * n_out) + 8.0 * n_in * n_out * D * D + kb + kg
        return {"bytes": by, "flops": 2 * (enc + mac + mb * n_in + mg * n_out)}
    T, hd, nq = case["tokens"], case["head_dim"], case["queries"]
    nj = hd + T - 1
    ks, ms = _switch(case, L, T - 1)
    ko, mo = _switch(case, L, hd - 1, hd - 1)
    kr, mr = _switch(case, L, T, T)
    ka, ma = _switch(case, L - 2, nj - 1)
    by = row * (2 * L * (nq + 2) + 2 * (L - 2) * nq + 2 * (L - 3) * nq) + 3 * ks + ko + kr / T + ka
    corr = n * 2.0 * L * (hd * math.log2(hd) * nq + 2 * hd * math.log2(2 * hd))
    fl = ms * (nq + 2) + nq * (mo + mr + ma) + corr + nq * (4.0 * L * n * T + 4.0 * (L - 2) * n * nj)
    return {"bytes": by, "flops": 2 * fl}


def tolerance(case):
    """Residues are whole numbers and agree bit for bit.  A client's decoded slots are fp64: against the definition they
    are off by 6.6e-16, in whatever order the sums run.  With real slots the imaginary part is only the encryption
    noise, 1e-10 to 1e-7 of the slots, so the same absolute error is up to 1e-6 of its norm."""
    if case["kind"] != "client":
        return "exact"
    return {"rel": 3e-15 if case["imag"] else 5e-6, "max": 1e-13 if case["imag"] else 2e-4, "differ": 0.0}


def exact(case, seed):
    """The decoded slots of a client case from the definition: the canonical embedding of the rounded coefficients plus
    the encryption error (with real slots the imaginary part is noise and has no value of its own).  Every other
    output is whole residues, which are compared bit for bit."""
    if case["kind"] != "client":
        return None
    _, re, im, _, e = _client_inputs(case, seed)
    z = re.cpu().numpy() + 1j * (0.0 if im is None else im.cpu().numpy())
    n = 1 << case["log_n"]
    M, scale = n // 2, 2.0 ** case["scale_log2"]
    s = np.empty(M, dtype=np.int64)                        # slot j sits at 5^j = 4 s + 1 modulo 2N
    p = 1
    for j in range(M):
        s[j] = (p - 1) // 4
        p = p * 5 % (2 * n)
    y = np.empty(M, dtype=np.complex128)
    y[s] = z
    zeta = np.exp(-1j * np.pi * np.arange(M) / n)
    v = zeta * np.fft.fft(y) * (scale * 2.0 / n)
    m = np.concatenate([v.real, v.imag])
    m = np.copysign(np.floor(np.abs(m) + 0.5), m) + e.cpu().numpy()
    w = np.fft.ifft((m[:M] + 1j * m[M:]) / zeta)[s] * (M / scale)
    return {"pt": None, "ct": None, "back": None, "re": w.real.copy(),
            "im": w.imag.copy() if case["imag"] else None}
