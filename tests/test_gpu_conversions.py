"""Base conversions fused into the column pass that follows them (N >= 2^13), over
what their units and tables depend on: one to eight sources, cut-short last
digits, one to four targets in a unit, narrow and wide primes on either side,
each scheme.  Compared with the oracle limb for limb.
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


def params(q_bits, p_bits, alpha, log_n, scheme="ckks"):
    w = dict(q_bits=q_bits, p_bits=p_bits, log_nmax=16, log_n=log_n, alpha=alpha, scheme=scheme,
             t=65537 if scheme != "ckks" else 0)
    if scheme == "bfv":
        w.update(b_bits=[60] * (len(q_bits) + 1), msk_bits=60)
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


W, M, S = 60, 45, 30  # a wide prime, a narrow one, a small narrow one


@pytest.mark.parametrize("log_n,q_bits,p_bits,alpha,nl", [
    (13, [W] + [M] * 4, [W] * 4, 4, 5),       # one source in the last digit
    (13, [W] + [M] * 4, [W] * 4, 4, 1),       # no narrow target
    (13, [W] + [M] * 7, [W], 1, 8),           # digits of one limb, full and part units
    (13, [W] + [M] * 8, [W] * 2, 2, 9),
    (14, [W] + [M] * 9, [W] * 3, 3, 8),
    (14, [W] + [M] * 10, [W] * 5, 5, 11),     # five sources in tables of eight
    (14, [M] * 12, [M] * 8, 8, 12),           # no wide prime
    (13, [S] * 6 + [W] * 3, [M, W], 3, 9),    # small primes, wide ones last
    (15, [W] + [M] * 12, [W] * 4, 8, 13),
    (16, [W] + [M] * 8, [W] * 4, 4, 9),
    (13, [W] * 6 + [M] * 2, [W] * 2, 4, 8),   # too many wide targets for the fused lift
    (13, [W] * 6, [W] * 2, 2, 5),             # wide primes alone, more than one a digit
    (13, [W] * 5, [W], 1, 5),
])
def test_ckks(log_n, q_bits, p_bits, alpha, nl):
    p = params(q_bits, p_bits, alpha, log_n)
    ctx = context(p)
    a, b, key = draws(p, 100 * len(q_bits) + nl + log_n)
    a, b = a[:, :nl], b[:, :nl]
    a[1, :, 1::2] = np.array(p.q[:nl], dtype=np.uint64)[:, None] - np.uint64(1)  # residues at the top of their range
    print("conversions: N=2^%d, %s | %s, alpha=%d, level %d" % (log_n, q_bits, p_bits, alpha, nl), flush=True)
    ca, cb = C.Ciphertext(a, 1.0), C.Ciphertext(b, 1.0)
    want = C.hmult_relin(ca, cb, key, p)
    m = ctx.hmult_relin(dev(a), dev(b), dev(key))
    assert np.array_equal(host(m), want.data)
    g = C.galois_element(7, p.n)
    assert np.array_equal(host(ctx.rotate(dev(a), g, dev(key))), C.rotate(ca, g, key, p).data)
    out = dev(b)
    ctx.keyswitch(dev(a[1]), dev(key), out, accumulate=True)
    ks = C.keyswitch(a[1], key, p)
    assert np.array_equal(host(out), np.stack([C.poly_add(b[c], ks[c], p.q[:nl]) for c in range(2)]))
    if nl >= 2:
        scaled = C.rescale(want, p).data
        assert np.array_equal(host(ctx.rescale(m)), scaled)
        flat = m.clone()  # in place: the result over the front of the operand
        ctx.rescale(flat, out=flat.view(-1)[:scaled.size].view(2, nl - 1, p.n))
        assert np.array_equal(host(flat).reshape(-1)[:scaled.size].reshape(scaled.shape), scaled)


@pytest.mark.parametrize("bits,k,alpha", [(M, 2, 2), (M, 1, 1), (55, 1, 1), (55, 2, 2)])
def test_bgv(bits, k, alpha):
    p = params([W] + [bits] * 4, [W] * k, alpha, 13, "bgv")
    ctx = context(p)
    a, b, key = draws(p, bits + k)
    want = G.hmult_relin(G.Ciphertext(a), G.Ciphertext(b), key, p)
    m = ctx.hmult_relin(dev(a), dev(b), dev(key))
    assert np.array_equal(host(m), want.data)
    assert np.array_equal(host(ctx.modswitch(m)), G.modswitch(want, p).data)


@pytest.mark.parametrize("bits,k,alpha", [(M, 2, 2), (M, 1, 1), (55, 1, 1), (55, 2, 2)])
def test_bfv(bits, k, alpha):
    # the product's key switch takes coefficients, the rotation's an NTT
    p = params([bits] * 4, [W] * k, alpha, 13, "bfv")
    ctx = context(p)
    a, b, key = draws(p, bits + k)
    assert np.array_equal(host(ctx.hmult_relin(dev(a), dev(b), dev(key))), F.hmult_relin(a, b, key, p))
    g = C.galois_element(3, p.n)
    assert np.array_equal(host(ctx.rotate(dev(a), g, dev(key))), F.rotate(a, g, key, p))


# bases of every kind in one plan: fused from up to 4 and 8 sources, converted by
# its own launch (wide primes, two a digit), 2 to 5 special primes
def test_batch_of_every_kind():
    from paper_2503_22227_amd import BatchPlan
    items = []
    for i, (log_n, q_bits, p_bits, alpha, nl) in enumerate([
            (13, [W] + [M] * 4, [W] * 4, 4, 5), (13, [W] * 6, [W] * 2, 2, 5), (13, [W] + [M] * 9, [W] * 5, 5, 8),
            (14, [M] * 12, [M] * 8, 8, 12), (13, [W] * 5, [W], 1, 4)]):
        p = params(q_bits, p_bits, alpha, log_n)
        a, b, key = draws(p, 40 + i)
        items.append((context(p), dev(a[:, :nl]), dev(b[:, :nl]), dev(key)))
    outs = [torch.empty_like(a) for _, a, _, _ in items]
    plan = BatchPlan([(c, a, b, k, o) for (c, a, b, k), o in zip(items, outs)])
    want = [host(c.hmult_relin(a, b, k)) for c, a, b, k in items]
    for grid in (0, 7):
        for stage in range(13):
            plan.set_grid(stage, grid)
        for o in outs:
            o.zero_()
        print("batch of every kind, grid %d" % grid, flush=True)
        plan.run(graph=False)
        assert all(np.array_equal(host(o), w) for o, w in zip(outs, want))


# steps above and below the size from which wide limbs keep the large tile
@pytest.mark.parametrize("count", [1, 40])
def test_batch_tiles(count):
    from paper_2503_22227_amd import BatchPlan
    p = params([W] + [M] * 2, [W] * 4, 2, 16)
    ctx = context(p)
    a, b, key = (dev(x) for x in draws(p, 9))
    outs = [torch.zeros_like(a) for _ in range(count)]
    plan = BatchPlan([(ctx, a, b, key, o) if i % 2 else (ctx, a, a, key, o) for i, o in enumerate(outs)])
    print("batch of %d items" % count, flush=True)
    plan.run(graph=False)
    want = [host(ctx.hmult_relin(a, a, key)), host(ctx.hmult_relin(a, b, key))]
    assert all(np.array_equal(host(o), want[i % 2]) for i, o in enumerate(outs))
