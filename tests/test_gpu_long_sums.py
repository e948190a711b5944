"""Key switches of many digits at N = 2^12, where the inner product on a special prime
below 2^46 is a sum of FP64 products: constant polynomials make every product the
largest there is, of one sign, so the sum grows by q / 2 a digit.  Compared with the
oracle."""
import numpy as np
import pytest

from oracle import ckks as C
from oracle import params as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# one digit short of a reduction of the sum, that digit, one more, and many
@pytest.mark.parametrize("limbs", [31, 32, 33, 50])
def test_special_prime_sum(limbs):
    from paper_2503_22227_amd import Context
    p = P.make_params(dict(scheme="ckks", log_n=12, log_nmax=12, q_bits=[40] * limbs, p_bits=[46], alpha=1, t=0))
    assert 2 ** 45 < p.p[0] < 2 ** 46
    ctx = Context(p.q, p.p, p.log_n, p.alpha, log_nmax=p.log_nmax)
    d = np.ones((limbs, p.n), dtype=np.uint64)  # the constant 1: 1 in every extension
    key = np.zeros((limbs, 2, limbs + 1, p.n), dtype=np.uint64)
    key[:, 0, :] = 1
    key[:, 0, limbs] = (p.p[0] - 1) // 2
    key[:, 1, limbs] = (p.p[0] + 1) // 2
    dev = lambda x: torch.from_numpy(x.view(np.int64)).cuda()  # noqa: E731
    out = torch.zeros(2, limbs, p.n, dtype=torch.int64, device="cuda")
    print("sum of %d digits" % limbs, flush=True)
    ctx.keyswitch(dev(d), dev(key), out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint64), np.stack(C.keyswitch(d, key, p)))
