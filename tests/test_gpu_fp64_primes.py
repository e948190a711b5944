"""Primes on both sides of the FP64 bound (2^46) in one chain.

Transforms of primes below 2^46 run in FP64, the others in 64-bit integers,
and the steps between them (base conversions, lifts, tails) join the two.  The
chain here mixes the largest primes below 2^46, the smallest above, small
ones (20 and 30 bits) and 60-bit ones, so a dropped or converted limb of either
kind meets targets of either kind.  Whole numbers, compared with the oracle
limb for limb, on uniform residues and on the extreme ones (0 and q - 1).
"""
import numpy as np
import pytest

import synthetic
from oracle import ckks as C
from oracle import params as P
from oracle.ntt import intt, ntt

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BOUND = 1 << 46


def near_bound(count, step):
    """The ``count`` primes = 1 mod 2^17 closest to the bound, below (step -1) or above it (step 1)."""
    out, c = [], (BOUND // (1 << 17)) * (1 << 17) + 1
    c -= (1 << 17) if step < 0 and c >= BOUND else 0
    while len(out) < count:
        if P.is_prime(c) and (c < BOUND) == (step < 0):
            out.append(c)
        c += step * (1 << 17)
    return out


def params(log_n, order):
    below, above = near_bound(3, -1), near_bound(2, 1)
    used = set()
    wide = P.next_primes_down(60, 1 << 17, 4, used)
    small = P.next_primes_down(20, 1 << 17, 1, used) + P.next_primes_down(30, 1 << 17, 1, used)
    pool = {"b": below, "a": above, "w": wide[:2], "s": small}
    q = [pool[k].pop(0) for k in order]
    return P.Params(log_n, 16, q, wide[2:], 3)


def context(p):
    from paper_2503_22227_amd import Context
    return Context(p.q, p.p, p.log_n, p.alpha, log_nmax=p.log_nmax)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().view(np.uint64)


def residues(rng, moduli, n):
    """Uniform residues, the first 64 and last 64 extreme (0 or q - 1)."""
    out = synthetic.uniform_residues(rng, moduli, n)
    for i, m in enumerate(moduli):
        for at in (slice(0, 64), slice(n - 64, n)):
            out[i, at] = rng.integers(0, 2, 64).astype(np.uint64) * np.uint64(m - 1)
    return out


@pytest.mark.parametrize("log_n", [12, 13, 14, 15, 16])
def test_transforms(log_n):
    p = params(log_n, "bwasba")
    ctx = context(p)
    moduli = p.q + p.p
    rng = np.random.default_rng(log_n)
    print("fp64 transforms at log_n=%d" % log_n, flush=True)
    full = np.stack([np.full(p.n, m - 1, dtype=np.uint64) for m in moduli])
    for x in (residues(rng, moduli, p.n), full):
        for tiles in (0, 1 << 20):  # 4096-residue tiles, small tiles
            ctx.set_tuning(0, {"ntt_small_below": tiles})
            f = host(ctx.ntt(dev(x), 0, len(moduli)))
            b = host(ctx.intt(dev(x), 0, len(moduli)))
            for i, m in enumerate(moduli):
                assert np.array_equal(f[i], ntt(x[i], m, p.psi(m))), (log_n, i, tiles)
                assert np.array_equal(b[i], intt(x[i], m, p.psi(m))), (log_n, i, tiles)


# the dropped limb and the digits' limbs: below / above the bound, small, wide
@pytest.mark.parametrize("log_n,order", [(12, "wbasb"), (13, "bwsab"), (13, "babsw"), (14, "wbbsa"), (15, "sabwb"),
                                         (16, "wabbs")])
def test_operations(log_n, order):
    p = params(log_n, order)
    ctx = context(p)
    rng = np.random.default_rng(100 + log_n)
    print("fp64 operations at log_n=%d, order %s" % (log_n, order), flush=True)
    qp = p.q + p.p
    key = np.stack([np.stack([residues(rng, qp, p.n) for _ in range(2)]) for _ in range(p.dnum())])
    a, b = (np.stack([residues(rng, p.q, p.n) for _ in range(2)]) for _ in range(2))
    g = C.galois_element(5, p.n)
    for fused in (0, 1 << 20):
        ctx.set_tuning(0, {"ntt_small_below": fused, "ntt_fused_small_below": fused})
        for nl in (len(p.q), len(p.q) - 1, 2):
            ca, cb = C.Ciphertext(a[:, :nl], 1.0), C.Ciphertext(b[:, :nl], 1.0)
            m = ctx.hmult_relin(dev(a[:, :nl]), dev(b[:, :nl]), dev(key))
            want = C.hmult_relin(ca, cb, key, p)
            assert np.array_equal(host(m), want.data), (nl, fused)
            assert np.array_equal(host(ctx.rescale(m)), C.rescale(want, p).data), (nl, fused)
            assert np.array_equal(host(ctx.rotate(dev(a[:, :nl]), g, dev(key))), C.rotate(ca, g, key, p).data), (nl, fused)
