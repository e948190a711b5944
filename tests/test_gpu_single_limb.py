"""Key switch and rescale at N = 2^12, where a workgroup holds a whole limb and
the steps between the transforms run inside them, over the shapes of its index
arithmetic: digits larger than the basis, cut-short and single digits, one to
eight special primes, each scheme.  Compared with the oracle limb for limb.
"""
import numpy as np
import pytest

import synthetic
from oracle import bfv as F
from oracle import bgv as G
from oracle import ckks as C
from oracle import params as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def params(limbs, k, alpha, scheme="ckks", bits=45):
    w = dict(q_bits=[60] + [bits] * (limbs - 1), p_bits=[60] * k, log_nmax=16, log_n=12, alpha=alpha, scheme=scheme,
             t=65537 if scheme != "ckks" else 0)
    if scheme == "bfv":
        w.update(b_bits=[60] * (limbs + 1), msk_bits=60)
    return P.make_params(w)


def context(p):
    from paper_2503_22227_amd import Context
    return Context(p.q, p.p, p.log_n, p.alpha, log_nmax=p.log_nmax, scheme=p.scheme, t=p.t, b=p.b, m_sk=p.msk)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().view(np.uint64)


def draws(p, seed):
    rng = np.random.default_rng(seed)
    ct = lambda: np.stack([synthetic.uniform_residues(rng, p.q, p.n) for _ in range(2)])  # noqa: E731
    key = np.stack([np.stack([synthetic.uniform_residues(rng, p.q + p.p, p.n) for _ in range(2)])
                    for _ in range(p.dnum())])
    return ct(), ct(), key


# limbs, special primes, alpha, level: alpha above the whole basis, a digit per
# limb, a last digit of one limb, eight sources and eight special primes
@pytest.mark.parametrize("limbs,k,alpha,nl", [(3, 1, 8, 3), (3, 1, 8, 1), (4, 1, 5, 4), (5, 2, 1, 4), (9, 3, 4, 9),
                                              (9, 8, 8, 9), (24, 4, 8, 24), (24, 5, 3, 17)])
def test_ckks(limbs, k, alpha, nl):
    p = params(limbs, k, alpha)
    ctx = context(p)
    a, b, key = draws(p, limbs * 100 + nl)
    a, b = a[:, :nl], b[:, :nl]
    print("single limb: %d limbs, k=%d, alpha=%d, level %d" % (limbs, k, alpha, nl), flush=True)
    ca, cb = C.Ciphertext(a, 1.0), C.Ciphertext(b, 1.0)
    want = C.hmult_relin(ca, cb, key, p)
    m = ctx.hmult_relin(dev(a), dev(b), dev(key))
    assert np.array_equal(host(m), want.data)
    g = C.galois_element(7, p.n)
    assert np.array_equal(host(ctx.rotate(dev(a), g, dev(key))), C.rotate(ca, g, key, p).data)
    # key switch on its own, added to what is there
    out = dev(b)
    ctx.keyswitch(dev(a[1]), dev(key), out, accumulate=True)
    ks = C.keyswitch(a[1], key, p)
    mod = p.q[:nl]
    assert np.array_equal(host(out), np.stack([C.poly_add(b[c], ks[c], mod) for c in range(2)]))
    if nl >= 2:
        scaled = C.rescale(want, p).data
        assert np.array_equal(host(ctx.rescale(m)), scaled)
        flat = m.clone()  # in place: the result over the front of the operand
        ctx.rescale(flat, out=flat.view(-1)[:scaled.size].view(2, nl - 1, p.n))
        assert np.array_equal(host(flat).reshape(-1)[:scaled.size].reshape(scaled.shape), scaled)


@pytest.mark.parametrize("bits", [45, 55])
def test_bgv(bits):
    p = params(5, 2, 2, "bgv", bits)
    ctx = context(p)
    a, b, key = draws(p, bits)
    want = G.hmult_relin(G.Ciphertext(a), G.Ciphertext(b), key, p)
    m = ctx.hmult_relin(dev(a), dev(b), dev(key))
    assert np.array_equal(host(m), want.data)
    assert np.array_equal(host(ctx.modswitch(m)), G.modswitch(want, p).data)


def test_bfv():
    p = params(4, 1, 2, "bfv", 55)
    ctx = context(p)
    a, b, key = draws(p, 5)
    assert np.array_equal(host(ctx.hmult_relin(dev(a), dev(b), dev(key))), F.hmult_relin(a, b, key, p))
    g = C.galois_element(3, p.n)
    assert np.array_equal(host(ctx.rotate(dev(a), g, dev(key))), F.rotate(a, g, key, p))
