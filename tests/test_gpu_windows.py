"""Standalone transforms of windows of a chain with wide and narrow primes: any
first limb, both classes, over the 4096-residue tiles' launches.  Compared with the
oracle limb for limb, and one launch a pass whatever the classes' order."""
import numpy as np
import pytest

import synthetic
from oracle import ntt as T
from oracle import params as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

_CTX = {}


def context(log_n):
    from paper_2503_22227_amd import Context
    if log_n not in _CTX:
        p = P.make_params(dict(scheme="ckks", log_n=log_n, log_nmax=16, q_bits=[60, 45, 45, 60, 45, 60, 60, 45],
                               p_bits=[45, 60], alpha=2, t=0))
        c = Context(p.q, p.p, p.log_n, p.alpha, log_nmax=p.log_nmax)
        c.set_tuning(0, dict(c.get_tuning(1), ntt_small_below=0))
        _CTX[log_n] = (p, c)
    return _CTX[log_n]


# the whole chain, its end, one limb of either class, runs of one class, all odd starts
@pytest.mark.parametrize("log_n", [13, 14, 15, 16])
@pytest.mark.parametrize("first,count,polys", [(0, 10, 1), (1, 9, 2), (3, 5, 3), (1, 2, 2), (5, 2, 1), (7, 1, 2),
                                               (9, 1, 1), (2, 8, 1), (0, 3, 2)])
def test_window(log_n, first, count, polys):
    from paper_2503_22227_amd import _lib
    p, ctx = context(log_n)
    moduli = (p.q + p.p)[first:first + count]
    rng = np.random.default_rng(1000 * log_n + 100 * first + count)
    x = np.stack([synthetic.uniform_residues(rng, moduli, p.n) for _ in range(polys)])
    d = torch.from_numpy(x.view(np.int64)).cuda()
    print("window %d + %d, %d polynomials, N=2^%d" % (first, count, polys, log_n), flush=True)
    _lib.profile_enable(True)
    ctx.ntt(d, first, count, polys)
    torch.cuda.synchronize()
    launches = _lib.profile_read()
    _lib.profile_enable(False)
    got = d.cpu().numpy().view(np.uint64)
    for c in range(polys):
        for i, q in enumerate(moduli):
            assert np.array_equal(got[c, i], T.ntt(x[c, i], q, p.psi(q))), (c, i)
    assert sorted(n for n, _ in launches.values()) == [1, 1], launches
    ctx.intt(d, first, count, polys)
    torch.cuda.synchronize()
    assert np.array_equal(d.cpu().numpy().view(np.uint64), x)
