"""Work that a program using this framework has it do, as cases that can be timed.

Each case is one pass through the public entry points (``Context``,
``BatchPlan``, ``pdq.GpuExecutor``) on inputs made from a seed.  The sizes are
those of the workloads in ``synthetic``, of the tests and of the benchmark:
ring degrees 2^12 to 2^16 and 2 to 24 limbs of the 60 + 23 x 45-bit chain with
four 60-bit special primes (digits of 4 or 8 primes), the small 60 + 40-bit
chain, and the 14 x 55-bit chain of the exact schemes.

Contexts (tables derived from the primes alone) are made once per shape and
shared by the states, as a program keeps one context for all its ciphertexts;
every ciphertext, key and plan belongs to a state.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2503_22227_amd import BatchPlan, Context, pdq
from paper_2503_22227_amd.params import chain_for

DEVICE = "cuda"

# q_bits, p_bits, largest ring degree, auxiliary base bits (BFV)
CHAINS = {
    "main": dict(q_bits=[60] + [45] * 23, p_bits=[60] * 4, log_nmax=16),
    "small": dict(q_bits=[60, 40], p_bits=[60], log_nmax=12),
    "exact": dict(q_bits=[55] * 14, p_bits=[60], log_nmax=15, b_bits=[60] * 14, msk_bits=60),
}
T_PLAIN = 65537
LOG_SCALE = 40

_CONTEXTS = {}


def listed():
    return [
        # the smallest call: one product and its rescale in the smallest ring (launches and latency)
        dict(name="mult_n12_l2", kind="mult", chain="small", log_n=12, limbs=2, alpha=1),
        # a rotation in a small ring at a low, odd level
        dict(name="rotate_n13_l5_a4", kind="rotate", chain="main", log_n=13, limbs=5, alpha=4),
        # an ordinary product in a mid-size ring, the last digit cut short
        dict(name="mult_n14_l11_a8", kind="mult", chain="main", log_n=14, limbs=11, alpha=8),
        # the query circuit's usual product: the serving chain some way down its levels
        dict(name="mult_n16_l9_a4", kind="mult", chain="main", log_n=16, limbs=9, alpha=4),
        # the benchmark's product and rescale, and its rotation, at the full level
        dict(name="mult_n16_l24_a8", kind="mult", chain="main", log_n=16, limbs=24, alpha=8),
        dict(name="rotate_n16_l24_a8", kind="rotate", chain="main", log_n=16, limbs=24, alpha=8),
        # exact integers: the BEHZ product, and a BGV product with its modulus switch lower down
        dict(name="bfv_mult_n15_l14", kind="bfv_mult", chain="exact", log_n=15, limbs=14, alpha=1),
        dict(name="bgv_mult_n15_l9", kind="bgv_mult", chain="exact", log_n=15, limbs=9, alpha=1),
        # the client: slots to a ciphertext, and a ciphertext back to slots
        dict(name="encrypt_n16_l24", kind="encrypt", chain="main", log_n=16, limbs=24, alpha=4),
        dict(name="decrypt_n16_l17", kind="decrypt", chain="main", log_n=16, limbs=17, alpha=4),
        # many ciphertexts of mixed ring degree and level in one plan, replayed as a graph
        dict(name="batch_64", kind="batch", chain="main", items=64, log_n_low=14, log_n=16, low=4, limbs=24, alpha=8,
             shape_seed=7),
        # a whole private-table query (some 300 operations over all levels)
        dict(name="query_n16_r100", kind="query", chain="main", log_n=16, limbs=24, alpha=4, rows=100),
    ]


def draw(rng: random.Random):
    kind = rng.choice(["mult", "mult", "rotate", "rotate", "bgv_mult", "bfv_mult", "encrypt", "decrypt", "batch",
                       "query"])
    log_n = rng.randint(12, 16)
    alpha = rng.choice([4, 8])
    # over the logarithm of the level, so that the low levels, where a program spends most operations, come often
    limbs = min(24, int(round(2.0 * 12.0 ** rng.random())))
    if kind in ("bgv_mult", "bfv_mult"):
        n_q = 14
        c = dict(kind=kind, chain="exact", log_n=rng.randint(13, 15), limbs=n_q, alpha=1)
        if kind == "bgv_mult":
            c["limbs"] = min(n_q, int(round(2.0 * 7.0 ** rng.random())))
        return c
    if kind == "batch":
        low = rng.randint(2, 6)
        return dict(kind=kind, chain="main", items=int(round(3 * 12.0 ** rng.random())), log_n_low=rng.randint(13, 15),
                    log_n=rng.randint(15, 16), low=low, limbs=rng.randint(low + 2, 24), alpha=8,
                    shape_seed=rng.randint(0, 1 << 20))
    if kind == "query":
        # the circuit needs the whole chain's levels, and four columns of the padded rows in N / 2 slots
        log_n = rng.randint(13, 16)
        return dict(kind=kind, chain="main", log_n=log_n, limbs=24, alpha=4, rows=rng.randint(10, 127))
    if kind in ("encrypt", "decrypt"):
        return dict(kind=kind, chain="main", log_n=log_n, limbs=limbs, alpha=4)
    return dict(kind=kind, chain="main", log_n=log_n, limbs=limbs, alpha=alpha)


def context(case, log_n=None) -> Context:
    log_n = case["log_n"] if log_n is None else log_n
    scheme = {"bfv_mult": "bfv", "bgv_mult": "bgv"}.get(case["kind"], "ckks")
    key = (scheme, case["chain"], log_n, case["alpha"])
    if key not in _CONTEXTS:
        w = dict(CHAINS[case["chain"]])
        if scheme != "bfv":
            w.pop("b_bits", None)
        ch = chain_for(w)
        _CONTEXTS[key] = Context(ch["q"], ch["p"], log_n, case["alpha"], log_nmax=w["log_nmax"], scheme=scheme,
                                 t=0 if scheme == "ckks" else T_PLAIN, b=ch["b"] if scheme == "bfv" else (),
                                 m_sk=ch["msk"] if scheme == "bfv" else 0)
    return _CONTEXTS[key]


# ---------------------------------------------------------------- inputs
def generator(seed: int) -> torch.Generator:
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def residues(gen, moduli, n, *lead, out=None):
    """Uniform residues [*lead, len(moduli), n]: what ciphertexts and keys look like to anyone without the secret."""
    out = torch.empty(*lead, len(moduli), n, dtype=torch.int64, device=DEVICE) if out is None else out
    flat = out.view(-1, len(moduli), n)
    for i, m in enumerate(moduli):
        flat[:, i] = torch.randint(0, int(m), (flat.shape[0], n), generator=gen, device=DEVICE, dtype=torch.int64)
    return out


def switch_key(gen, ctx):
    return residues(gen, ctx.q + ctx.p, ctx.n, ctx.dnum, 2)


def small(gen, n, bound):
    return torch.randint(-bound, bound + 1, (n,), generator=gen, device=DEVICE, dtype=torch.int64)


def gaussian(gen, n):
    """Rounded normal errors, sigma 3.2, cut at 19."""
    e = torch.randn(n, generator=gen, device=DEVICE, dtype=torch.float64) * 3.2
    return e.round().clamp(-19, 19).to(torch.int64)


def slots(gen, n):
    """Complex slots with parts uniform in [-1, 1]."""
    return torch.view_as_complex(torch.rand(n // 2, 2, generator=gen, device=DEVICE, dtype=torch.float64) * 2 - 1)


def batch_shapes(case):
    """(log_n, limbs) of the items; limb counts and degrees uniform over their ranges."""
    r = random.Random(case["shape_seed"])
    return [(r.randint(case["log_n_low"], case["log_n"]), r.randint(case["low"], case["limbs"]))
            for _ in range(case["items"])]


def message(case, seed):
    """Of a decryption: the message coefficients and the error that went into the ciphertext."""
    n = 1 << case["log_n"]
    gen = generator(seed)
    m = torch.randn(n, generator=gen, device=DEVICE, dtype=torch.float64) * (2.0 ** LOG_SCALE / math.sqrt(n))
    return gen, m.round().to(torch.int64), gaussian(gen, n)


def prepare(case, seed):
    kind, s = case["kind"], {"kind": case["kind"]}
    if kind == "batch":
        gen = generator(seed)
        shapes = batch_shapes(case)
        ctxs = {ln: context(case, ln) for ln in sorted({x[0] for x in shapes})}
        keys = {ln: switch_key(gen, c) for ln, c in ctxs.items()}
        sizes = [2 * nl << ln for ln, nl in shapes]
        out = torch.empty(sum(sizes), dtype=torch.int64, device=DEVICE)
        items, at = [], 0
        for (ln, nl), size in zip(shapes, sizes):
            c = ctxs[ln]
            a, b = (residues(gen, c.q[:nl], c.n, 2) for _ in range(2))
            items.append((c, a, b, keys[ln], out[at:at + size].view(2, nl, c.n)))
            at += size
        s.update(plan=BatchPlan(items), out=out)
        return s
    ctx = context(case)
    nl = case["limbs"]
    q = ctx.q[:nl]
    s["ctx"] = ctx
    if kind == "decrypt":
        gen, m, e = message(case, seed)
        s["sk"] = ctx.key_ntt(small(gen, ctx.n, 1))
        s["ct"] = ctx.encrypt(m, e, residues(gen, q, ctx.n), s["sk"])
        return s
    gen = generator(seed)
    if kind == "encrypt":
        s.update(z=slots(gen, ctx.n), e=gaussian(gen, ctx.n), mask=residues(gen, q, ctx.n),
                 sk=ctx.key_ntt(small(gen, ctx.n, 1)))
    elif kind == "rotate":
        s.update(a=residues(gen, q, ctx.n, 2), key=switch_key(gen, ctx))
        s["galois"] = ctx.galois_element(int(seed) % (ctx.n // 2 - 1) + 1)
    elif kind == "query":
        ops, outs, _ = pdq.plan_query(ctx.q, nl, 2.0 ** 45, case["rows"], int(seed) % 4, (int(seed) // 4 + 1) % 4)
        keys = {"rlk": switch_key(gen, ctx)}
        for r in pdq.rotation_amounts(ops):
            keys[r] = switch_key(gen, ctx)
        s.update(ops=ops, outs=outs, last=pdq.last_uses(ops, outs), run=pdq.GpuExecutor(ctx, keys),
                 inputs={k: residues(gen, q, ctx.n, 2) for k in ("T", "LO", "HI")})
    else:
        s.update(a=residues(gen, q, ctx.n, 2), b=residues(gen, q, ctx.n, 2), key=switch_key(gen, ctx))
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    kind = s["kind"]
    if kind == "batch":
        s["plan"].run(graph=True)
        return s["out"]
    ctx = s["ctx"]
    if kind == "mult":
        prod = ctx.hmult_relin(s["a"], s["b"], s["key"])
        return {"product": prod, "rescaled": ctx.rescale(prod)}
    if kind == "rotate":
        return ctx.rotate(s["a"], s["galois"], s["key"])
    if kind == "bfv_mult":
        return ctx.hmult_relin(s["a"], s["b"], s["key"])
    if kind == "bgv_mult":
        prod = ctx.hmult_relin(s["a"], s["b"], s["key"])
        return {"product": prod, "switched": ctx.modswitch(prod)}
    if kind == "encrypt":
        m = ctx.encode(s["z"], 2.0 ** LOG_SCALE)
        return {"message": m, "ciphertext": ctx.encrypt(m, s["e"], s["mask"], s["sk"])}
    if kind == "decrypt":
        coeffs = ctx.crt_centered(ctx.decrypt(s["ct"], s["sk"]), 2.0 ** LOG_SCALE)
        return {"coefficients": coeffs, "slots": ctx.decode(coeffs)}
    # the serving loop's way through an op list: registers freed after their last use
    regs = dict(s["inputs"])
    for i, op in enumerate(s["ops"]):
        s["run"].step(op, regs)
        for r in [x for x in op[2:] if isinstance(x, str)] + [op[1]]:
            if s["last"].get(r, -1) <= i:
                regs.pop(r, None)
    return [regs[name] for name in s["outs"]]


# ---------------------------------------------------------------- what a pass cannot do without
def transforms(log_n, count):
    """Modular multiplications of `count` limb transforms."""
    return count * log_n << (log_n - 1)


def key_switch(log_n, nl, alpha, k):
    """(64-bit words, modular multiplications) of one key switch: the key's limbs of this level read once;
    transforms of the digits, their extension and the special limbs, base conversions, products."""
    dn = -(-nl // alpha)
    ext = sum(nl + k - min(alpha, nl - j * alpha) for j in range(dn))
    conv = sum(min(alpha, nl - j * alpha) * (nl + k - min(alpha, nl - j * alpha)) for j in range(dn))
    n = 1 << log_n
    words = 2 * dn * (nl + k) * n
    mults = transforms(log_n, nl + ext + 2 * k + 2 * nl) + n * (conv + 2 * dn * (nl + k) + 2 * k * nl + 2 * nl)
    return words, mults


def op_work(op, log_n, nl, alpha, k):
    n = 1 << log_n
    if op == "mult":
        w, f = key_switch(log_n, nl, alpha, k)
        return w + 6 * nl * n, f + 4 * nl * n
    if op == "rotate":
        w, f = key_switch(log_n, nl, alpha, k)
        return w + 4 * nl * n, f
    if op == "rescale":
        return (4 * nl - 2) * n, transforms(log_n, 2 * nl) + 2 * nl * n
    return 6 * nl * n, 2 * nl * n  # element-wise


def work(case):
    kind, log_n, nl, alpha = case["kind"], case["log_n"], case["limbs"], case["alpha"]
    k = len(CHAINS[case["chain"]]["p_bits"])
    n = 1 << log_n
    if kind == "mult" or kind == "bgv_mult":
        todo = [op_work("mult", log_n, nl, alpha, k), op_work("rescale", log_n, nl, alpha, k)]
    elif kind == "rotate":
        todo = [op_work("rotate", log_n, nl, alpha, k)]
    elif kind == "bfv_mult":
        b = len(CHAINS[case["chain"]]["b_bits"]) + 1
        w, f = op_work("mult", log_n, nl, alpha, k)
        # 7 polynomials through the extended basis, the conversions to and from the auxiliary base
        todo = [(w, f + transforms(log_n, 7 * (nl + b) + 2 * nl) + n * (4 * nl * b + 3 * nl * b + 3 * b * nl))]
    elif kind == "batch":
        shapes = batch_shapes(case)
        todo = [op_work("mult", ln, l, alpha, k) for ln, l in shapes]
        # one key for all items of a ring degree
        most = {ln: max(l for x, l in shapes if x == ln) for ln, _ in shapes}
        todo += [(-key_switch(ln, l, alpha, k)[0], 0) for ln, l in shapes]
        todo += [(key_switch(ln, l, alpha, k)[0], 0) for ln, l in most.items()]
    elif kind == "query":
        ops, outs, regs = pdq.plan_query(chain_for(CHAINS[case["chain"]])["q"], nl, 2.0 ** 45, case["rows"], 0, 1)
        todo = [op_work({"hmult": "mult", "rot": "rotate", "rescale": "rescale"}.get(op[0], "add"), log_n,
                        regs[op[2]][0] if op[2] in regs else regs[op[1]][0] if op[1] in regs else nl, alpha, k)
                for op in ops]
        # over the whole query the ciphertexts may stay on the chip: its inputs, each key once, its outputs
        amounts = len(pdq.rotation_amounts(ops)) + 1
        words = 3 * 2 * nl * n + amounts * key_switch(log_n, nl, alpha, k)[0] + sum(2 * regs[r][0] * n for r in outs)
        todo = [(0, f) for _, f in todo] + [(words, 0)]
    elif kind == "encrypt":
        todo = [((2 + 1 + 4 * nl) * n, transforms(log_n, nl) + 2 * nl * n + 4 * (log_n << (log_n - 1)))]
    else:
        todo = [((4 * nl + 2) * n, transforms(log_n, nl) + nl * n + nl * (nl - 1) // 2 * n + 4 * (log_n << (log_n - 1)))]
    return {"bytes": 8.0 * sum(w for w, _ in todo), "flops": 2.0 * sum(f for _, f in todo)}


# ---------------------------------------------------------------- the computed numbers, without the library
def exact(case, seed):
    """Decryption ends in computed numbers: the ciphertext's phase is the message plus its error, whole numbers
    far below the modulus, so the coefficients are known, and the slots follow by a Fourier transform taken here
    in extended precision.  Everything else is whole numbers."""
    if case["kind"] != "decrypt":
        return None
    n = 1 << case["log_n"]
    _, m, e = message(case, seed)
    x = (m + e).cpu().numpy().astype(np.longdouble) / np.longdouble(2.0 ** LOG_SCALE)
    turn = np.exp(1j * np.arctan2(np.longdouble(0), np.longdouble(-1)) * np.arange(n, dtype=np.longdouble) / n)
    values = np.fft.ifft(x * turn) * n  # the polynomial at the odd powers of the primitive 2N-th root
    at = np.empty(n // 2, dtype=np.int64)
    p = 1
    for j in range(n // 2):
        at[j] = (p - 1) // 2
        p = p * 5 % (2 * n)
    return {"coefficients": x.astype(np.float64), "slots": values[at].astype(np.complex128)}
