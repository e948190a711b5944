"""The ModUp conversion in a launch of its own, which bases of wide primes alone with
more than one prime a digit take: every limb grouping, coefficients scaled by the
INTT (CKKS, batches) and given by the caller (BFV), short last digits.  Compared with
the oracle limb for limb."""
import numpy as np
import pytest

import synthetic
from oracle import bfv as F
from oracle import ckks as C
from oracle import params as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def setup(scheme, log_n, limbs, alpha, seed):
    from paper_2503_22227_amd import Context
    w = dict(scheme=scheme, log_n=log_n, log_nmax=16, q_bits=[60] * limbs, p_bits=[60] * 2, alpha=alpha,
             t=65537 if scheme == "bfv" else 0)
    if scheme == "bfv":
        w.update(b_bits=[60] * (limbs + 1), msk_bits=60)
    p = P.make_params(w)
    rng = np.random.default_rng(seed)
    a, b = (np.stack([synthetic.uniform_residues(rng, p.q, p.n) for _ in range(2)]) for _ in range(2))
    key = np.stack([np.stack([synthetic.uniform_residues(rng, p.q + p.p, p.n) for _ in range(2)])
                    for _ in range(p.dnum())])
    return p, Context(p.q, p.p, p.log_n, p.alpha, log_nmax=p.log_nmax, scheme=scheme, t=p.t, b=p.b, m_sk=p.msk), a, b, key


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().view(np.uint64)


def conversions(fn):
    """Launches of the conversion's own kernel while fn runs."""
    from paper_2503_22227_amd import _lib
    _lib.profile_enable(True)
    out = fn()
    torch.cuda.synchronize()
    r = _lib.profile_read()
    _lib.profile_enable(False)
    return out, sum(n for k, (n, _) in r.items() if k.endswith("modup_bconv"))


@pytest.mark.parametrize("chunk", [4, 8, 16])
@pytest.mark.parametrize("scheme,log_n,limbs,alpha", [("ckks", 13, 10, 2), ("ckks", 14, 7, 4), ("bfv", 13, 5, 2)])
def test_single(scheme, log_n, limbs, alpha, chunk):
    p, ctx, a, b, key = setup(scheme, log_n, limbs, alpha, log_n + limbs)
    ctx.set_tuning(0, dict(ctx.get_tuning(1), modup_chunk=chunk))
    print("chunk %d %s N=2^%d limbs %d alpha %d" % (chunk, scheme, log_n, limbs, alpha), flush=True)
    got, n = conversions(lambda: ctx.hmult_relin(dev(a), dev(b), dev(key)))
    assert n == 1
    want = (F.hmult_relin(a, b, key, p) if scheme == "bfv"
            else C.hmult_relin(C.Ciphertext(a, 1.0), C.Ciphertext(b, 1.0), key, p).data)
    assert np.array_equal(host(got), want)
    ctx.close()


@pytest.mark.parametrize("chunk", [4, 8, 16])
def test_batch(chunk):
    from paper_2503_22227_amd import BatchPlan
    items, want = [], []
    for log_n, limbs, alpha, nl in ((13, 10, 2, 10), (13, 10, 2, 3), (14, 7, 4, 7), (13, 6, 8, 6)):
        p, ctx, a, b, key = setup("ckks", log_n, limbs, alpha, 50 + nl)
        items.append((ctx, dev(a[:, :nl]), dev(b[:, :nl]), dev(key), torch.zeros(2, nl, p.n, dtype=torch.int64, device="cuda")))
        want.append(C.hmult_relin(C.Ciphertext(a[:, :nl], 1.0), C.Ciphertext(b[:, :nl], 1.0), key, p).data)
    plan = BatchPlan(items)
    plan.set_modup_chunk(chunk)
    assert plan.stage_units(3) > 0
    for grid in (0, 9):
        plan.set_grid(3, grid)
        print("batch chunk %d grid %d" % (chunk, grid), flush=True)
        _, n = conversions(plan.run)
        assert n == 1
        for it, w in zip(items, want):
            assert np.array_equal(host(it[4]), w)
            it[4].zero_()
    plan.close()
