"""Launches of wide primes alone just below and from the size on which they take
4096-residue tiles: standalone transforms of windows; and levels of wide primes
alone in a chain that has narrow ones.  Compared with the oracle limb for limb."""
import numpy as np
import pytest

import synthetic
from oracle import ckks as C
from oracle import ntt as T
from oracle import params as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

_CTX = {}


def context(log_n, limbs):
    from paper_2503_22227_amd import Context
    p = P.make_params(dict(scheme="ckks", log_n=log_n, log_nmax=16, q_bits=[60] * limbs, p_bits=[59] * 4, alpha=8, t=0))
    c = Context(p.q, p.p, p.log_n, p.alpha, log_nmax=p.log_nmax)
    c.set_tuning(0, dict(c.get_tuning(1), ntt_small_below=0, ntt_fused_small_below=0))
    return p, c


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().view(np.uint64)


# (first limb, limbs, polynomials): one limb short of the size and the size, with
# another prime than limb 0's, in one, two and more polynomials
@pytest.mark.parametrize("log_n,window", [(16, (1, 31, 1)), (16, (2, 16, 2)), (15, (3, 21, 3)), (15, (1, 16, 4)),
                                          (14, (0, 32, 4)), (14, (5, 18, 7)), (13, (3, 25, 5)), (13, (1, 32, 4))])
def test_windows(log_n, window):
    first, count, polys = window
    if log_n not in _CTX:
        _CTX[log_n] = context(log_n, 33)
    p, ctx = _CTX[log_n]
    moduli = (p.q + p.p)[first:first + count]
    rng = np.random.default_rng(log_n * 100 + count)
    x = np.stack([synthetic.uniform_residues(rng, moduli, p.n) for _ in range(polys)])
    d = dev(x)
    print("wide window %s N=2^%d" % (window, log_n), flush=True)
    ctx.ntt(d, first, count, polys)
    got = host(d)
    for c in range(polys):
        for i, q in enumerate(moduli):
            assert np.array_equal(got[c, i], T.ntt(x[c, i], q, p.psi(q))), (c, i)
    ctx.intt(d, first, count, polys)
    assert np.array_equal(host(d), x)


# a level whose Q-limbs are of wide primes alone, in a chain that has narrow ones:
# among the special primes too, or not; large and small tiles of the fused passes
@pytest.mark.parametrize("fused_small", [0, 4096])
@pytest.mark.parametrize("log_n,p_bits", [(13, [60, 45]), (14, [60] * 3), (15, [45] * 2), (16, [60, 59])])
def test_wide_level(log_n, p_bits, fused_small):
    from paper_2503_22227_amd import Context
    p = P.make_params(dict(scheme="ckks", log_n=log_n, log_nmax=16, q_bits=[60] * 5 + [45] * 2, p_bits=p_bits, alpha=2,
                           t=0))
    ctx = Context(p.q, p.p, p.log_n, p.alpha, log_nmax=p.log_nmax)
    ctx.set_tuning(0, dict(ctx.get_tuning(1), ntt_fused_small_below=fused_small))
    nl = 5
    rng = np.random.default_rng(7 * log_n + fused_small)
    a, b = (np.stack([synthetic.uniform_residues(rng, p.q[:nl], p.n) for _ in range(2)]) for _ in range(2))
    key = np.stack([np.stack([synthetic.uniform_residues(rng, p.q + p.p, p.n) for _ in range(2)])
                    for _ in range(p.dnum())])
    print("wide level N=2^%d | %s fused_small %d" % (log_n, p_bits, fused_small), flush=True)
    dk = dev(key)
    want = C.hmult_relin(C.Ciphertext(a, 1.0), C.Ciphertext(b, 1.0), key, p)
    m = ctx.hmult_relin(dev(a), dev(b), dk)
    assert np.array_equal(host(m), want.data)
    g = C.galois_element(5, p.n)
    assert np.array_equal(host(ctx.rotate(dev(a), g, dk)), C.rotate(C.Ciphertext(a, 1.0), g, key, p).data)
    assert np.array_equal(host(ctx.rescale(m)), C.rescale(want, p).data)
