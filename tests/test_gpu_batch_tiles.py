"""Batches around the sizes where a launch's wide limbs change tiles, which each ring
degree decides for itself: bases of wide primes alone, converted by a launch of
their own or (digits of one limb) in the column pass, and mixed ones.  Every item
equals the single operation, which other tests compare with the oracle."""
import numpy as np
import pytest

import synthetic
from oracle import params as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def item(log_n, q_bits, p_bits, alpha, seed):
    from paper_2503_22227_amd import Context
    p = P.make_params(dict(scheme="ckks", q_bits=q_bits, p_bits=p_bits, log_nmax=16, log_n=log_n, alpha=alpha, t=0))
    rng = np.random.default_rng(seed)
    dev = lambda x: torch.from_numpy(x.view(np.int64)).cuda()  # noqa: E731
    ct = [dev(np.stack([synthetic.uniform_residues(rng, p.q, p.n) for _ in range(2)])) for _ in range(2)]
    key = dev(np.stack([np.stack([synthetic.uniform_residues(rng, p.q + p.p, p.n) for _ in range(2)])
                        for _ in range(p.dnum())]))
    return Context(p.q, p.p, p.log_n, p.alpha, log_nmax=p.log_nmax), ct[0], ct[1], key


# the product's own limbs have 6 or 4 tiles of 4096 residues an item at N = 2^13: the
# counts put each list of a launch below and above 512
@pytest.mark.parametrize("q_bits,p_bits,alpha", [([60] * 3, [60] * 2, 2), ([60] * 3, [60], 1), ([60, 60, 45], [60] * 2, 2),
                                                 ([60, 45, 45], [45, 60, 60, 60], 4)])
@pytest.mark.parametrize("count", [1, 30, 85, 86])
def test_counts(q_bits, p_bits, alpha, count):
    from paper_2503_22227_amd import BatchPlan
    kinds = [item(13, q_bits, p_bits, alpha, 1), item(14, q_bits, p_bits, alpha, 2)]
    use = [kinds[0]] * count + [kinds[1]]  # and one item of another degree
    outs = [torch.zeros_like(it[1]) for it in use]
    plan = BatchPlan([(c, a, b, k, o) for (c, a, b, k), o in zip(use, outs)])
    want = [c.hmult_relin(a, b, k) for c, a, b, k in kinds]
    for grid in (0, 64):
        for stage in range(13):
            plan.set_grid(stage, grid)
        for o in outs:
            o.zero_()
        print("batch tiles %s | %s alpha %d count %d grid %d" % (q_bits, p_bits, alpha, count, grid), flush=True)
        plan.run(graph=False)
        torch.cuda.synchronize()
        for i, o in enumerate(outs):
            assert torch.equal(o, want[i // count])
    plan.close()
