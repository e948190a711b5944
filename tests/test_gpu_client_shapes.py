"""The client's fused passes at the shapes the workload tests do not reach.

Encoding and decoding run one FFT in two launches at every ring degree (an odd
and an even number of stages in each); encryption and decryption fold their
lift, product and copy into the passes of the transform, on small tiles for few
limbs and large ones for many; the CRT composition takes FP64 digits where
every limb but the first is below 2^46 and integer ones otherwise.  Whole
numbers are compared with the oracle exactly.  Decoding and the composition end
in doubles: log2 N stages, each rounding by at most a few 2^-53 of the largest
value, bound the error by 8 log2(N) 2^-53 times the largest sum.
"""
import numpy as np
import pytest

import synthetic
from oracle import ckks as C
from oracle import params as P
from oracle.rns import centered, crt, product

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def params(log_n, limbs, bits):
    w = dict(q_bits=[60] + [bits] * (limbs - 1), p_bits=[60], log_nmax=16, log_n=log_n, alpha=4, scheme="ckks")
    return P.make_params(w)


def context(p, scheme="ckks", t=0):
    from paper_2503_22227_amd import Context
    return Context(p.q, p.p, p.log_n, p.alpha, log_nmax=p.log_nmax, scheme=scheme, t=t)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("log_n,limbs,bits", [(12, 1, 45), (13, 2, 45), (14, 31, 45), (15, 9, 50), (16, 20, 45),
                                              (13, 17, 55)])
def test_encrypt_decrypt(log_n, limbs, bits):
    p = params(log_n, limbs, bits)
    ctx = context(p)
    st = synthetic.streams(log_n)
    rng = np.random.default_rng(limbs)
    print("client shapes log_n=%d limbs=%d bits=%d" % (log_n, limbs, bits), flush=True)
    s = synthetic.ternary(st["sk"], p.n)
    # coefficients over the whole signed range the entry point takes
    m = rng.integers(-(1 << 62), 1 << 62, p.n, dtype=np.int64)
    m[:4] = [0, -1, (1 << 62), -(1 << 62)]
    e = synthetic.gaussian(st["ct_e"], p.n)
    a = synthetic.uniform_residues(st["ct_a"], p.q, p.n)
    s_ntt = ctx.key_ntt(dev(s))
    ct = ctx.encrypt(dev(m), dev(e), dev(a.view(np.int64)), s_ntt)
    mod = p.q[:limbs]
    sh = C.small_to_ntt(s, mod, p)
    want = C.poly_add(C.poly_neg(C.poly_mul(a, sh, mod), mod),
                      C.small_to_ntt(m.astype(object) + e.astype(object), mod, p), mod)
    got = host(ct).view(np.uint64)
    assert np.array_equal(got[0], want) and np.array_equal(got[1], a)
    x = ctx.decrypt(ct, s_ntt)
    exact = m.astype(object) + e.astype(object)
    assert np.array_equal(host(x).view(np.uint64), np.stack([(exact % q).astype(np.uint64) for q in mod]))


@pytest.mark.parametrize("log_n,limbs,bits", [(12, 2, 45), (13, 8, 45), (13, 9, 45), (14, 16, 45), (13, 25, 45),
                                              (12, 31, 45), (13, 32, 45), (13, 5, 50), (12, 1, 45)])
def test_crt_composition(log_n, limbs, bits):
    p = params(log_n, limbs, bits)
    ctx = context(p)
    mod = p.q[:limbs]
    x = synthetic.uniform_residues(np.random.default_rng(limbs), mod, p.n)
    Q = product(mod)
    for i, q in enumerate(mod):  # the extremes: 0, Q - 1, the middle of the range from both sides
        x[i, :4] = [0, (Q - 1) % q, (Q // 2) % q, (Q // 2 + 1) % q]
    if Q.bit_length() > 1000:  # values that a double holds: the centred ones modulo 2^1000
        v = centered(crt(x, mod), Q)
        v = np.array([int(abs(c)) % (1 << 1000) * (1 if c >= 0 else -1) for c in v], dtype=object)
        x = np.stack([(v % q).astype(np.uint64) for q in mod])
    print("crt log_n=%d limbs=%d bits=%d" % (log_n, limbs, bits), flush=True)
    got = host(ctx.crt_centered(dev(x.view(np.int64)), 2.0 ** 40))
    want = centered(crt(x, mod), product(mod))
    # limbs roundings of the Horner sum, each at most 2^-53 of a partial sum no larger than the whole's bound
    for g, v in zip(got.tolist(), want.tolist()):
        w = v / 2 ** 40
        assert abs(g - w) <= 2 * limbs * 2.0 ** -53 * abs(w) + 2.0 ** -39 * (limbs == 1), (g, w)


@pytest.mark.parametrize("log_n", [12, 13, 14, 15, 16])
def test_encode_decode(log_n):
    p = params(log_n, 2, 45)
    ctx = context(p)
    rng = np.random.default_rng(log_n)
    z = synthetic.complex_slots(rng, p.n // 2)
    print("fft log_n=%d" % log_n, flush=True)
    m = host(ctx.encode(dev(z), 2.0 ** 40))
    want = C.encode(z, 2.0 ** 40, p.n)
    d = np.abs(m.astype(object) - want)
    assert max(d) <= 1 and (d != 0).mean() < 0.01
    x = rng.uniform(-1, 1, p.n)
    out = host(ctx.decode(dev(x)))
    ref = np.fft.ifft(x.astype(np.longdouble) * np.exp(1j * np.pi * np.arange(p.n, dtype=np.longdouble) / p.n)) * p.n
    at = (C._slot_exponents(p.n) - 1) // 2
    bound = 8 * log_n * 2.0 ** -53 * float(np.abs(ref).max())
    assert np.abs(out - ref[at].astype(np.complex128)).max() <= bound
