// N = 2^12: transforms of a whole limb in one workgroup, and the key switch and
// rescale built from them.
//
// 1024 threads hold 4 residues each and run six radix-4 rounds through 34 KiB
// of LDS, every twiddle of a thread fetched together with its residues.  A limb of
// a wide prime is bound by the integer issue of the one CU it has: 24576
// butterflies of about 30 instructions, 4.8 us.
//
// A launch of this size costs its latency, on the device and on the host, so
// the steps between the transforms ride in them: a key switch is four launches
// (nine before) and a rescale one (four): HMult+Relin and rescale of two 60 and
// 40-bit limbs took 78.3 us in 13 launches and take 61.9 in five.
#include <hip/hip_runtime.h>

#include "ks_dev.hpp"
#include "ntt_dev.hpp"

namespace rf {

constexpr int kSLog = 12, kSN = 1 << kSLog, kSE = 4, kSThreads = kSN / kSE;
constexpr int kSWords = kSN + kSN / 16;

// The transform of the limb pro gives, its residue p of thread t's at p = t +
// 1024 r; results by out(p, value) (forward: unreduced in FP64, in [0, q) in
// integers; inverse: the last stage's).  lds may be reused after a barrier.
template <typename Ar, bool FWD, typename Pro, typename Out>
__device__ __forceinline__ void single_ntt(uint64_t *lds, const TwPair *__restrict__ tw_all, const Ar &ar,
                                           const Pro &pro, const Out &out) {
    const auto *tw = twiddles<Ar>(tw_all);
    const LimbLds L{lds};
    const int t = threadIdx.x;
    typename Ar::V v[kSE];
    typename Ar::Tw twc[tw_slots(kSLog, kSE)];
#pragma unroll
    for (int r = 0; r < kSE; ++r) v[r] = pass_in(pro, t + r * kSThreads, ar);
    ntt_rounds<Ar, kSLog, FWD, !FWD, 0, kSE, kTwPrefetch>(L, t, 1u, tw, ar, twc);
#pragma unroll
    for (int r = 0; r < kSE; ++r) L(t + r * kSThreads) = Ar::bits(v[r]);
    __syncthreads();
    ntt_rounds<Ar, kSLog, FWD, !FWD, 0, kSE, kTwCached>(L, t, 1u, tw, ar, twc);
#pragma unroll
    for (int r = 0; r < kSE; ++r) {
        typename Ar::V x = Ar::raw(L(t + r * kSThreads));
        if constexpr (FWD && !Ar::kFp) x = csub(csub(x, ar.q2), ar.q);
        out((size_t)(t + r * kSThreads), x);
    }
}

// The same with the arithmetic of prime g; an Epi (forward) or the canonical
// store into `to` (inverse).
template <typename Pro, typename Epi>
__device__ __forceinline__ void single_fwd(uint64_t *lds, const TwPair *tw, const PrimeConst &pc, bool fp,
                                           const Pro &pro, const Epi &epi) {
    if (fp) {
        const ArFp ar(pc);
        single_ntt<ArFp, true>(lds, tw, ar, pro, [&](size_t p, double x) { epi.fp(p, x, ar.f); });
    } else {
        const ArInt ar(pc);
        single_ntt<ArInt, true>(lds, tw, ar, pro, [&](size_t p, uint64_t x) { epi(p, x); });
    }
}

template <typename Pro>
__device__ __forceinline__ void single_inv(uint64_t *lds, const TwPair *tw, const PrimeConst &pc, bool fp,
                                           const Pro &pro, uint64_t *to) {
    if (fp) {
        const ArFp ar(pc);
        single_ntt<ArFp, false>(lds, tw, ar, pro, [&](size_t p, double x) { to[p] = ar.canon_last(x); });
    } else {
        const ArInt ar(pc);
        single_ntt<ArInt, false>(lds, tw, ar, pro, [&](size_t p, uint64_t x) { to[p] = ar.canon_last(x); });
    }
}

// Limbs of a batch, any polynomials.
template <bool FWD>
__global__ __launch_bounds__(kSThreads) void ntt_single_kernel(NttBatch b, FpMask fpm, const TwPair *__restrict__ tw_all,
                                                               const PrimeConst *__restrict__ pcs) {
    __shared__ uint64_t lds[kSWords];
    const uint32_t li = blockIdx.x / b.n_polys, poly = blockIdx.x - li * b.n_polys;
    const uint32_t g = b.pmap ? b.pmap[li] : b.prime_base + li;
    const PrimeConst pc = pcs[g];
    const LoadPro pro{b.in + (size_t)poly * b.in_poly_stride + ((size_t)li << kSLog)};
    uint64_t *out = b.out + (size_t)poly * b.out_poly_stride + ((size_t)li << kSLog);
    const TwPair *tw = tw_all + ((size_t)g << kSLog);
    if constexpr (FWD) single_fwd(lds, tw, pc, fpm.has(g), pro, StoreEpi{out});
    else single_inv(lds, tw, pc, fpm.has(g), pro, out);
}

struct SingleArgs {
    const uint64_t *a, *b, *d, *evk;
    uint64_t *dc, *ext, *ip, *out;
    const TwPair *tw_fwd, *tw_inv;
    const PrimeConst *pcs, *pcs_mu, *pcs_md;
    const uint64_t *modup, *md_cross, *md_negp, *pinv;
    size_t modup_stride;
    IpFold fold;
    uint32_t nl, L, K, alpha, dn;
};

// INTT of the polynomial to switch, limb i, with its digit's input factor.
__global__ __launch_bounds__(kSThreads) void single_first_kernel(SingleArgs a, FpMask fpm) {
    __shared__ uint64_t lds[kSWords];
    const uint32_t i = blockIdx.x;
    const PrimeConst pc = a.pcs_mu[i];
    const size_t li = (size_t)i << kSLog, poly = (size_t)a.nl << kSLog;
    const TwPair *tw = a.tw_inv + li;
    uint64_t *to = a.dc + li;
    const bool fp = fpm.has(i);
    if (a.fold.mode == 1)
        single_inv(lds, tw, pc, fp, TensorPro{a.fold.a + poly + li, a.fold.b + poly + li, pc.q, pc.r64, pc.r64_p, pc.one_p}, to);
    else if (a.fold.mode == 2) single_inv(lds, tw, pc, fp, GatherPro{a.fold.a + poly + li, a.fold.galois, kSLog}, to);
    else single_inv(lds, tw, pc, fp, LoadPro{a.d + li}, to);
}

// ModUp conversion of a digit (source limbs x, s of them) to one target, as the
// prologue of the target's NTT.  factor non-null: x is unscaled.
struct ModupPro {
    static constexpr bool kBlocked = false;
    const uint64_t *x, *factor, *cross;
    const PrimeConst *src;  // the sources' constants
    uint32_t s, narrow;     // narrow: bit i set if source i is below kFpPrimeBound
    uint64_t q, r64, r64_p, one_p;
    __device__ __forceinline__ uint64_t y(uint32_t i, size_t idx) const {
        const uint64_t v = x[((size_t)i << kSLog) + idx];
        return factor ? shoup(v, factor[2 * i], factor[2 * i + 1], src[i].q) : v;
    }
    __device__ __forceinline__ uint64_t operator()(size_t idx) const {
        MacAcc acc;
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)kMaxAlpha; ++i)
            if (i < s) acc.mac(y(i, idx), cross[i]);
        return reduce128_lazy(acc.value(), q, r64, r64_p, one_p);
    }
    __device__ __forceinline__ double fp(size_t idx, const FpMod &f) const {
        double acc = 0.0;
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)kMaxAlpha; ++i)
            if (i < s) {
                const double c = FpMod::from_u52(cross[i]);
                const uint64_t v = y(i, idx);
                if ((narrow >> i) & 1) {
                    acc += f.mul(FpMod::from_u52(v), c);
                } else {  // a wide residue from its halves
                    acc += f.mul(FpMod::from_u52(v & 0x3fffffffu), c) +
                           f.mul(FpMod::from_u52(v >> 30), f.mul(1073741824.0, c));
                }
            }
        return acc;
    }
};

// Extension limb blockIdx.x: digits back to back, each its targets in the order
// of Q_l u P without the digit's own primes.
template <bool COEF>
__global__ __launch_bounds__(kSThreads) void single_modup_kernel(SingleArgs a, FpMask fpm) {
    __shared__ uint64_t lds[kSWords];
    const uint32_t per = a.nl + a.K - a.alpha;  // targets of a full digit
    const uint32_t last = a.dn - 1;
    const uint32_t jf = per ? blockIdx.x / per : last, j = jf < last ? jf : last, tt = blockIdx.x - j * per;
    const uint32_t start = j * a.alpha, s = min(a.alpha, a.nl - start);
    const uint32_t g = tt < start ? tt : (tt < a.nl - s ? tt + s : a.L + (tt - (a.nl - s)));
    const PrimeConst pc = a.pcs[g];
    const uint64_t *blk = a.modup + ((size_t)j * a.alpha + (s - 1)) * a.modup_stride;
    ModupPro pro;
    pro.x = (COEF ? a.d : a.dc) + ((size_t)start << kSLog);
    pro.factor = COEF ? blk : nullptr;
    pro.cross = blk + 2 * a.alpha + (size_t)g * a.alpha;
    pro.src = a.pcs + start;
    pro.s = s;
    pro.narrow = 0;
    for (uint32_t i = 0; i < s; ++i) pro.narrow |= fpm.has(start + i) ? 1u << i : 0u;
    pro.q = pc.q;
    pro.r64 = pc.r64;
    pro.r64_p = pc.r64_p;
    pro.one_p = pc.one_p;
    single_fwd(lds, a.tw_fwd + ((size_t)g << kSLog), pc, fpm.has(g), pro,
               StoreEpi{a.ext + ((size_t)blockIdx.x << kSLog)});
}

// Inner product sum_j ext_j evk_{j,c} on special limb a, as the prologue of its INTT.
struct IpPro {
    static constexpr bool kBlocked = false;
    const uint64_t *ext, *key;  // at the limb; digit strides below
    size_t key_stride;
    uint32_t dn, nl, K, alpha;
    uint64_t q, r64, r64_p, one_p;
    // special limb m - nl is target m - s of a digit of s primes
    __device__ __forceinline__ uint64_t src(uint32_t j, size_t idx) const {
        const uint32_t s = min(alpha, nl - j * alpha);
        return ext[(((size_t)j * (nl + K - alpha) - s) << kSLog) + idx];
    }
    __device__ __forceinline__ uint64_t operator()(size_t idx) const {
        u128 acc{0, 0};
#pragma unroll 2
        for (uint32_t j = 0; j < dn; ++j) mac(acc, src(j, idx), key[j * key_stride + idx]);
        return csub(reduce128_lazy(acc, q, r64, r64_p, one_p), 2 * q);
    }
    __device__ __forceinline__ double fp(size_t idx, const FpMod &f) const {
        double acc = 0.0;
        // 32 digits at a time: below 33 * 0.75 q < 2^51, red's range
        for (uint32_t j0 = 0; j0 < dn; j0 += 32) {
            const uint32_t j1 = min(dn, j0 + 32);
#pragma unroll 2
            for (uint32_t j = j0; j < j1; ++j)
                acc += f.mul(FpMod::from_u52(src(j, idx)), FpMod::from_u52(key[j * key_stride + idx]));
            acc = f.red(acc);
        }
        return acc;
    }
};

// Workgroups [0, 2K): special limb blockIdx.x / 2 of polynomial blockIdx.x & 1,
// with its INTT (the ModDown input factor folded in); the rest: the Q-limbs,
// 1024 coefficients each, leaving as ip P^-1 + addend (inner_product_unit).
__global__ __launch_bounds__(kSThreads) void single_ip_kernel(SingleArgs a, FpMask fpm) {
    __shared__ uint64_t lds[kSWords];
    const uint32_t w = blockIdx.x;
    if (w < 2 * a.K) {
        const uint32_t c = w & 1, k = w >> 1, g = a.L + k, m = a.nl + k;
        const PrimeConst pc = a.pcs_md[g];
        IpPro pro;
        pro.ext = a.ext + ((size_t)m << kSLog);
        const size_t key_poly = (size_t)(a.L + a.K) << kSLog;
        pro.key = a.evk + c * key_poly + ((size_t)g << kSLog);
        pro.key_stride = 2 * key_poly;
        pro.dn = a.dn;
        pro.nl = a.nl;
        pro.K = a.K;
        pro.alpha = a.alpha;
        pro.q = pc.q;
        pro.r64 = pc.r64;
        pro.r64_p = pc.r64_p;
        pro.one_p = pc.one_p;
        single_inv(lds, a.tw_inv + ((size_t)g << kSLog), pc, fpm.has(g), pro,
                   a.ip + (((size_t)c * (a.nl + a.K) + m) << kSLog));
        return;
    }
    const uint32_t u = w - 2 * a.K;
    // inner_product_unit takes blocks of kEw coefficients: threads 256 b.. are block b
    inner_product_unit<1>(a.d, a.ext, a.evk, a.ip, a.pcs, kSLog, a.nl, a.L, a.K, a.alpha, 4 * (u & 3), u >> 2, a.fold);
}

// ModDown of limb i of polynomial c: conversion, NTT, tail.
template <int KP>
__global__ __launch_bounds__(kSThreads) void single_moddown_kernel(SingleArgs a, FpMask fpm) {
    __shared__ uint64_t lds[kSWords];
    const uint32_t c = blockIdx.x & 1, i = blockIdx.x >> 1;
    const PrimeConst pc = a.pcs[i];
    ModdownPro<KP> pro;
    pro.src = a.ip + (((size_t)c * (a.nl + a.K) + a.nl) << kSLog);
    pro.stride = kSN;
    pro.K = a.K;
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        pro.half[k] = k < (int)a.K ? a.pcs[a.L + k].q >> 1 : 0;
        pro.cross[k] = k < (int)a.K ? a.md_cross[(size_t)i * a.K + k] : 0;
    }
    pro.negp = a.md_negp[i];
    pro.q = pc.q;
    pro.r64 = pc.r64;
    pro.r64_p = pc.r64_p;
    pro.one_p = pc.one_p;
    const ModdownFoldEpi epi{a.ip + (((size_t)c * (a.nl + a.K) + i) << kSLog), a.out + (((size_t)c * a.nl + i) << kSLog),
                             a.pinv[2 * i], a.pinv[2 * i + 1], pc.q};
    single_fwd(lds, a.tw_fwd + ((size_t)i << kSLog), pc, fpm.has(i), pro, epi);
}

// Division by the last prime, limb i of polynomial c: INTT of the last limb
// (again in every workgroup: a launch of its own costs as much), lift, NTT,
// tail.  The last limb passes through LDS, each thread's own residues.
template <bool KEEP_T>
__global__ __launch_bounds__(kSThreads) void single_divide_kernel(const uint64_t *in, uint64_t *out,
                                                                  const TwPair *__restrict__ tw_fwd,
                                                                  const TwPair *__restrict__ tw_inv,
                                                                  const PrimeConst *__restrict__ pcs,
                                                                  const uint64_t *__restrict__ tab, uint32_t nl,
                                                                  uint32_t L, FpMask fpm) {
    __shared__ uint64_t lds[kSWords];
    __shared__ uint64_t last[kSN];
    const uint32_t l = nl - 1, c = blockIdx.x & 1, i = blockIdx.x >> 1;
    const PrimeConst pl = pcs[l], pc = pcs[i];
    single_inv(lds, tw_inv + ((size_t)l << kSLog), pl, fpm.has(l), LoadPro{in + (((size_t)c * nl + l) << kSLog)}, last);
    __syncthreads();
    const uint64_t *t = tab + ((size_t)l * L + i) * 3;
    LiftPro<KEEP_T> pro;
    pro.last = last;
    pro.ql = pl.q;
    pro.ql_half = pl.q >> 1;
    pro.tinv = pl.tinv;
    pro.tinv_p = pl.tinv_p;
    pro.qld = pl.qd;
    pro.q = pc.q;
    pro.one_p = pc.one_p;
    pro.corr = t[2];
    pro.tmod = pc.tmod;
    pro.tmod_p = pc.tmod_p;
    const RescaleTailEpi epi{in + (((size_t)c * nl + i) << kSLog), out + (((size_t)c * l + i) << kSLog), t[0], t[1], pc.q};
    single_fwd(lds, tw_fwd + ((size_t)i << kSLog), pc, fpm.has(i), pro, epi);
}

static int check_launch(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RF_EHIP, std::string(what) + ": " + hipGetErrorString(e));
    return RF_OK;
}

int launch_ntt_single(const rf_ctx *c, const NttBatch &b, bool forward, hipStream_t s, const PrimeConst *pcs) {
    const dim3 g(b.per_poly * b.n_polys), t(kSThreads);
    ProfScope p(forward ? "ntt_fwd_single" : "ntt_inv_single", s);
    if (forward) hipLaunchKernelGGL(ntt_single_kernel<true>, g, t, 0, s, b, c->fp_mask, c->d_tw_fwd, pcs);
    else hipLaunchKernelGGL(ntt_single_kernel<false>, g, t, 0, s, b, c->fp_mask, c->d_tw_inv, pcs);
    return check_launch("NTT launch");
}

int launch_keyswitch_single(const rf_ctx *c, const IpFold &fold, const uint64_t *d, const uint64_t *coef,
                            const uint64_t *evk, uint64_t *dc, uint64_t *ext, uint64_t *ip, uint64_t *out,
                            uint32_t nl, hipStream_t s) {
    const uint64_t *md = c->scheme == RF_BGV ? c->d_moddown_t : c->d_moddown;
    SingleArgs a{};
    a.fold = fold;
    a.fold.pinv = a.pinv = c->d_moddown + moddown_pinv_off(c);
    a.d = d;
    a.evk = evk;
    a.dc = dc;
    a.ext = ext;
    a.ip = ip;
    a.out = out;
    a.tw_fwd = c->d_tw_fwd;
    a.tw_inv = c->d_tw_inv;
    a.pcs = c->d_pc;
    a.pcs_mu = pc_modup(c, nl);
    a.pcs_md = c->d_pc_md;
    a.modup = c->d_modup;
    a.modup_stride = c->modup_stride;
    a.md_cross = md + moddown_cross_off(c);
    a.md_negp = md + moddown_negp_off(c);
    a.nl = nl;
    a.L = c->L;
    a.K = c->K;
    a.alpha = c->alpha;
    a.dn = (nl + c->alpha - 1) / c->alpha;
    const dim3 t(kSThreads);
    int rc;
    const uint32_t ext_limbs = c->modup_levels[nl].ext_limbs;
    if (coef) {
        SingleArgs b = a;
        b.d = coef;
        ProfScope p("single_modup", s);
        hipLaunchKernelGGL(single_modup_kernel<true>, dim3(ext_limbs), t, 0, s, b, c->fp_mask);
    } else {
        {
            ProfScope p("single_first", s);
            hipLaunchKernelGGL(single_first_kernel, dim3(nl), t, 0, s, a, c->fp_mask);
        }
        ProfScope p("single_modup", s);
        hipLaunchKernelGGL(single_modup_kernel<false>, dim3(ext_limbs), t, 0, s, a, c->fp_mask);
    }
    {
        ProfScope p("single_ip", s);
        hipLaunchKernelGGL(single_ip_kernel, dim3(2 * c->K + 4 * nl), t, 0, s, a, c->fp_mask);
    }
    if ((rc = check_launch("key switch"))) return rc;
    ProfScope p("single_moddown", s);
    const dim3 g(2 * nl);
    switch (c->K) {
        case 1: hipLaunchKernelGGL(single_moddown_kernel<1>, g, t, 0, s, a, c->fp_mask); break;
        case 2: hipLaunchKernelGGL(single_moddown_kernel<2>, g, t, 0, s, a, c->fp_mask); break;
        case 3: hipLaunchKernelGGL(single_moddown_kernel<3>, g, t, 0, s, a, c->fp_mask); break;
        case 4: hipLaunchKernelGGL(single_moddown_kernel<4>, g, t, 0, s, a, c->fp_mask); break;
        default: hipLaunchKernelGGL(single_moddown_kernel<8>, g, t, 0, s, a, c->fp_mask); break;
    }
    return check_launch("ModDown");
}

int launch_divide_single(const rf_ctx *c, const uint64_t *in, uint64_t *out, uint32_t nl, bool keep_t, hipStream_t s) {
    ProfScope p("single_divide", s);
    const dim3 g(2 * (nl - 1)), t(kSThreads);
    if (keep_t)
        hipLaunchKernelGGL(single_divide_kernel<true>, g, t, 0, s, in, out, c->d_tw_fwd, c->d_tw_inv, c->d_pc,
                           c->d_rescale, nl, c->L, c->fp_mask);
    else
        hipLaunchKernelGGL(single_divide_kernel<false>, g, t, 0, s, in, out, c->d_tw_fwd, c->d_tw_inv, c->d_pc,
                           c->d_rescale, nl, c->L, c->fp_mask);
    return check_launch("rescale");
}

}  // namespace rf
