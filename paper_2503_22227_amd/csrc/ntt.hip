// Negacyclic NTT / INTT kernels of single operations; the device code is in
// ntt_dev.hpp (shared with the batched kernels).
#include <hip/hip_runtime.h>

#include "ntt_dev.hpp"

namespace rf {

struct LimbView {
    const uint64_t *in;
    uint64_t *out;
    uint32_t g;  // prime index
};

// grid.y runs over the limbs with the polynomials interleaved (limb li of every
// polynomial, then limb li + 1, ...): the tiles that share a prime's twiddles
// are launched back to back, 16 workgroups apart at N = 2^16, which places them
// on the same XCD (workgroups are dealt to the 8 XCDs in turn), so the second
// reads the twiddles from that XCD's L2.
//
// The limb index is uniform across the workgroup: held in a scalar register, so
// the prime map and the prime's constants are read with scalar loads instead of
// a vector load whose latency would delay the tile's own loads.
__device__ __forceinline__ LimbView limb_view(const NttBatch &b, int log_n, uint32_t limb) {
    const uint32_t li = __builtin_amdgcn_readfirstlane(limb / b.n_polys), poly = limb - li * b.n_polys;
    LimbView v;
    v.g = b.pmap ? b.pmap[li] : b.prime_base + li;
    v.in = b.in + (size_t)poly * b.in_poly_stride + ((size_t)li << log_n);
    v.out = b.out + (size_t)poly * b.out_poly_stride + ((size_t)li << log_n);
    return v;
}

// The limbs of a launch on tiles by class (ntt_cols_mixed): the wide ones first,
// since their workgroups take longest, N / 1024 workgroups each, then the narrow
// ones, N / 4096 each; polynomials interleaved.
struct MixGrid {
    LimbOrder o;
    uint32_t np;
};
struct MixUnit {
    uint32_t li, poly, g;
    int tile;
    bool fp;
};

template <int A, int B, bool COLS, typename Fp>
__device__ __forceinline__ MixUnit mix_unit(const MixGrid &m) {
    constexpr bool BIG = std::is_same_v<Fp, WideTiles>;
    constexpr int LOGN = A + B, TW = BIG ? LOGN - 12 : LOGN - 10, TN = LOGN - 12;
    MixUnit u;
    const uint32_t wide = m.o.n_wide * m.np;
    uint32_t w = blockIdx.x, e;
    u.fp = std::is_same_v<Fp, FpMask> && w >= wide << TW;
    if (u.fp) {
        w -= wide << TW;
        e = wide + (w >> TN);
        u.tile = w & ((1 << TN) - 1);
    } else {
        e = w >> TW;
        u.tile = w & ((1 << TW) - 1);
        if (COLS && !BIG) u.tile = xcd_grouped_tile<kMixTile, A>(u.tile, 1 << TW);
    }
    const uint32_t k = __builtin_amdgcn_readfirstlane(m.np == 1 ? e : m.np == 2 ? e >> 1 : e / m.np);
    u.poly = e - k * m.np;
    if (BIG && !m.o.ent) {
        u.li = k;
        u.g = m.o.base + k;
    } else {
        const uint32_t x = m.o.ent[u.fp ? k + m.o.gap : k];
        u.li = (x & 0xffffu) - m.o.base;
        u.g = x >> 16;
    }
    return u;
}

// The first `limbs` Q-limbs of np polynomials.
static MixGrid q_mix(const rf_ctx *c, uint32_t limbs, uint32_t np) {
    return MixGrid{c->order(c->q_order[limbs]), np};
}

// Grid of a launch of `limbs` limbs of each of np polynomials.
static dim3 mix_grid(const rf_ctx *c, uint32_t n_wide, uint32_t limbs, uint32_t np) {
    return dim3(np * (n_wide * (c->n / kMixTile) + (limbs - n_wide) * (c->n / kTile)));
}

// Transforms of wide limbs alone in the natural layout take 4096-residue tiles from
// two workgroups of them a CU on (half that at N = 2^13, where a 1024-residue tile
// of columns is half a line and no two of a line meet on an XCD).  Below, smaller
// tiles spread a launch over more CUs; from there on they only add twiddle loads
// and part lines.  Forward and inverse in tiles of 1024 against 4096: N = 2^16, 384
// tiles 48.3 and 54.8 us, 512 56.6 and 57.2, 768 74.1 and 70.2, 1536 127 and 118,
// 4096 313 and 266; N = 2^15, 512 57.6 and 58.2, 1024 88.8 and 83.8; N = 2^13, 192
// 32.4 and 32.8, 256 39.1 and 34.5.  The blocked passes, with a step of their own or
// whole lines in either tile, keep the small ones (768 tiles of a ModDown's rows 22.9
// and 25.8).
static uint32_t wide_tiles_from(const rf_ctx *c) { return c->log_n == 13 ? 256 : 512; }

template <int A, int B, bool FWD, bool BLK, typename Fp>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(ntt_waves(A)))) void ntt_cols_kernel(
    NttBatch b, Fp, MixGrid m, const TwPair *__restrict__ tw_all, const PrimeConst *__restrict__ pcs) {
    __shared__ uint64_t lds[(1 << A) * (kTile / (1 << A) + 1)];
    constexpr int LOGN = A + B;
    const MixUnit u = mix_unit<A, B, true, Fp>(m);
    const PrimeConst pc = pcs[u.g];
    ntt_cols_mixed<A, B, FWD, BLK, Fp>(lds, b.out + (size_t)u.poly * b.out_poly_stride + ((size_t)u.li << LOGN),
                              tw_all + ((size_t)u.g << LOGN), pc, u.fp, u.tile,
                              PlainPro<FWD>{b.in + (size_t)u.poly * b.in_poly_stride + ((size_t)u.li << LOGN)});
}

template <int A, int B, bool FWD, bool BLK, typename Fp>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(ntt_waves(B)))) void ntt_rows_kernel(
    NttBatch b, Fp, MixGrid m, const TwPair *__restrict__ tw_rows, const TwPair *__restrict__ tw_all,
    const PrimeConst *__restrict__ pcs) {
    __shared__ uint64_t lds[(1 << B) * (kTile / (1 << B) + 1)];
    constexpr int LOGN = A + B;
    const MixUnit u = mix_unit<A, B, false, Fp>(m);
    const PrimeConst pc = pcs[u.g];
    const size_t tl = (size_t)u.g << LOGN;
    ntt_rows_mixed<A, B, FWD, Fp>(lds, RowLoad<FWD, BLK>{b.in + (size_t)u.poly * b.in_poly_stride + ((size_t)u.li << LOGN)},
                              tw_rows + tl, tw_all + tl, pc, u.fp, u.tile,
                              RowStore<FWD, BLK>{b.out + (size_t)u.poly * b.out_poly_stride + ((size_t)u.li << LOGN)});
}

// First forward pass of NTT(conv) with the ModDown base conversion as its
// prologue: limb (c, i) of conv [2][nl][N] from the K P-limbs of ip[c].
template <int A, int B, int KP, typename Fp>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(KP == 8 ? 3 : kNttWavesFused))) void ntt_cols_moddown_kernel(
    Fp, MixGrid m, const uint64_t *ip, uint64_t *conv, const TwPair *__restrict__ tw_all, const PrimeConst *__restrict__ pcs,
    const uint64_t *__restrict__ cross, const uint64_t *__restrict__ negp, uint32_t nl, uint32_t L, uint32_t K) {
    __shared__ uint64_t lds[(1 << A) * (kTile / (1 << A) + 1)];
    constexpr int LOGN = A + B;
    const MixUnit u = mix_unit<A, B, true, Fp>(m);
    const uint32_t c = u.poly, i = u.li;
    const PrimeConst pc = pcs[i];
    const ModdownPro<KP> pro = moddown_pro<KP, LOGN>(ip, pcs, pc, cross, negp, c, i, nl, L, K);
    ntt_cols_mixed<A, B, true, true, Fp>(lds, conv + (((size_t)c * nl + i) << LOGN), tw_all + ((size_t)i << LOGN), pc, u.fp,
                               u.tile, pro);
}

// First forward pass of NTT(lift) with the rescale lift as its prologue: limb
// (c, i) of lift [2][l][N], l = nl - 1, from the last limb last[c].
template <int A, int B, bool KEEP_T, typename Fp>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kNttWavesFused))) void ntt_cols_lift_kernel(
    Fp, MixGrid m, const uint64_t *last, uint64_t *lift, const TwPair *__restrict__ tw_all, const PrimeConst *__restrict__ pcs,
    const uint64_t *__restrict__ tab, uint32_t nl, uint32_t L) {
    __shared__ uint64_t lds[(1 << A) * (kTile / (1 << A) + 1)];
    constexpr int LOGN = A + B;
    const uint32_t l = nl - 1;
    const MixUnit u = mix_unit<A, B, true, Fp>(m);
    const uint32_t c = u.poly, i = u.li;
    const PrimeConst pc = pcs[i];
    const LiftPro<KEEP_T> pro = lift_pro<KEEP_T, LOGN>(last, pcs, pc, tab, c, i, nl, L);
    ntt_cols_mixed<A, B, true, true, Fp>(lds, lift + (((size_t)c * l + i) << LOGN), tw_all + ((size_t)i << LOGN), pc, u.fp,
                               u.tile, pro);
}

// Last forward pass of NTT(conv) with the ModDown tail: limb (c, i) of conv
// [2][nl][N] -> out[c][i] = (ip[c][i] - NTT(conv)[c][i]) P^-1 (+ add_c[i]).
template <int A, int B, typename Fp>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(ntt_waves(B)))) void ntt_rows_moddown_kernel(
    Fp, MixGrid m, const uint64_t *conv, const TwPair *__restrict__ tw_rows, const TwPair *__restrict__ tw_all, const PrimeConst *__restrict__ pcs, const uint64_t *ip,
    uint64_t *out, const uint64_t *__restrict__ pinv, uint32_t nl, uint32_t K) {
    __shared__ uint64_t lds[(1 << B) * (kTile / (1 << B) + 1)];
    constexpr int LOGN = A + B;
    const MixUnit u = mix_unit<A, B, false, Fp>(m);
    const uint32_t c = u.poly, i = u.li;
    const PrimeConst pc = pcs[i];
    const ModdownFoldEpi epi{ip + (((size_t)c * (nl + K) + i) << LOGN), out + (((size_t)c * nl + i) << LOGN),
                             pinv[2 * i], pinv[2 * i + 1], pc.q};
    ntt_rows_mixed<A, B, true, Fp>(lds, BlkRawPro{conv + (((size_t)c * nl + i) << LOGN)}, tw_rows + ((size_t)i << LOGN),
                               tw_all + ((size_t)i << LOGN), pc, u.fp, u.tile, epi);
}

// First inverse pass of INTT(d2) with d2 = a1 b1 as its prologue: limb i of a, b
// ([2][nl][N], NTT domain); the row pass goes to dc [nl][N].
template <int A, int B, typename Fp>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(ntt_waves(B)))) void ntt_inv_rows_tensor_kernel(
    Fp, MixGrid m, const uint64_t *a, const uint64_t *b, uint64_t *dc, const TwPair *__restrict__ tw_rows, const TwPair *__restrict__ tw_all,
    const PrimeConst *__restrict__ pcs, uint32_t nl) {
    __shared__ uint64_t lds[(1 << B) * (kTile / (1 << B) + 1)];
    constexpr int LOGN = A + B;
    const MixUnit u = mix_unit<A, B, false, Fp>(m);
    const uint32_t i = u.li;
    const PrimeConst pc = pcs[i];
    const size_t li = (size_t)i << LOGN, poly = (size_t)nl << LOGN;
    const TensorPro pro{a + poly + li, b + poly + li, pc.q, pc.r64, pc.r64_p, pc.one_p};
    ntt_rows_mixed<A, B, false, Fp>(lds, pro, tw_rows + li, tw_all + li, pc, u.fp, u.tile, BlkRawEpi{dc + li});
}

// First inverse pass of INTT(sigma_g(a1)) with the automorphism as its
// prologue: limb i of a1 ([nl][N], NTT domain) permuted, row pass into dc.
template <int A, int B, typename Fp>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(ntt_waves(B)))) void ntt_inv_rows_gather_kernel(
    Fp, MixGrid m, const uint64_t *a1, uint64_t *dc, uint32_t galois, const TwPair *__restrict__ tw_rows, const TwPair *__restrict__ tw_all,
    const PrimeConst *__restrict__ pcs) {
    __shared__ uint64_t lds[(1 << B) * (kTile / (1 << B) + 1)];
    constexpr int LOGN = A + B;
    const MixUnit u = mix_unit<A, B, false, Fp>(m);
    const uint32_t i = u.li;
    const PrimeConst pc = pcs[i];
    const size_t li = (size_t)i << LOGN;
    const GatherPro pro{a1 + li, galois, (uint32_t)LOGN};
    ntt_rows_mixed<A, B, false, Fp>(lds, pro, tw_rows + li, tw_all + li, pc, u.fp, u.tile, BlkRawEpi{dc + li});
}

// Last forward pass of NTT(lift) with the rescale tail: limb (c, i) of lift
// [2][l][N] -> out[c][i] = (in[c][i] - NTT(lift)[c][i]) q_l^-1, l = nl - 1.
template <int A, int B, typename Fp>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(ntt_waves(B)))) void ntt_rows_rescale_kernel(
    Fp, MixGrid m, const uint64_t *lift, const TwPair *__restrict__ tw_rows, const TwPair *__restrict__ tw_all, const PrimeConst *__restrict__ pcs, const uint64_t *in,
    uint64_t *out, const uint64_t *__restrict__ tab, uint32_t nl, uint32_t L) {
    __shared__ uint64_t lds[(1 << B) * (kTile / (1 << B) + 1)];
    constexpr int LOGN = A + B;
    const uint32_t l = nl - 1;
    const MixUnit u = mix_unit<A, B, false, Fp>(m);
    const uint32_t c = u.poly, i = u.li;
    const PrimeConst pc = pcs[i];
    const uint64_t *t = tab + ((size_t)l * L + i) * 3;
    RescaleTailEpi epi{in + (((size_t)c * nl + i) << LOGN), out + (((size_t)c * l + i) << LOGN), t[0], t[1], pc.q};
    ntt_rows_mixed<A, B, true, Fp>(lds, BlkRawPro{lift + (((size_t)c * l + i) << LOGN)}, tw_rows + ((size_t)i << LOGN),
                               tw_all + ((size_t)i << LOGN), pc, u.fp, u.tile, epi);
}

template <int A, int B, bool FWD, bool COLS, int TILE, int E, bool BLK, typename Fp>
__global__ __launch_bounds__(TILE / E) void ntt_small_kernel(NttBatch b, Fp fpm, const TwPair *__restrict__ tw_all,
                                                             const PrimeConst *__restrict__ pcs) {
    constexpr int S = COLS ? (1 << A) : (1 << B);
    __shared__ uint64_t lds[S * (TILE / S + 1)];
    const LimbView v = limb_view(b, A + B, blockIdx.y);
    const PrimeConst pc = pcs[v.g];
    const TwPair *tw = tw_all + ((size_t)v.g << (A + B));
    if constexpr (COLS) ntt_cols_small<A, B, FWD, TILE, E, BLK>(lds, v.in, v.out, tw, pc, fpm.has(v.g), xcd_grouped_tile<TILE, A>(blockIdx.x, gridDim.x));
    else ntt_rows_small<A, B, FWD, TILE, E, BLK>(lds, v.in, v.out, tw, pc, fpm.has(v.g), blockIdx.x);
}

// Default residues per thread of the few-limb passes (4 measured faster than 8:
// the 8-limb inverse passes at N = 2^16 took 10.3 / 10.9 us against 10.8 / 12.7
// us); rf_tuning picks per level.
constexpr int kSmallE = 4;

// The passes of the fused ModDown, rescale and first-INTT launches on small
// tiles (the same prologues and epilogues as their 4096-tile kernels; natural
// twiddle tables, strict butterflies in both passes of a limb).
template <int A, int B, int TILE, int KP, typename Fp>
__global__ __launch_bounds__(TILE / kSmallE) void ntt_small_cols_moddown_kernel(
    Fp fpm, const uint64_t *ip, uint64_t *conv, const TwPair *__restrict__ tw_all, const PrimeConst *__restrict__ pcs,
    const uint64_t *__restrict__ cross, const uint64_t *__restrict__ negp, uint32_t nl, uint32_t L, uint32_t K) {
    __shared__ uint64_t lds[(1 << A) * (TILE / (1 << A) + 1)];
    constexpr int LOGN = A + B;
    const uint32_t c = blockIdx.y & 1, i = blockIdx.y >> 1;
    const PrimeConst pc = pcs[i];
    const ModdownPro<KP> pro = moddown_pro<KP, LOGN>(ip, pcs, pc, cross, negp, c, i, nl, L, K);
    ntt_cols_small_pro<A, B, true, TILE, kSmallE, true>(lds, pro, conv + (((size_t)c * nl + i) << LOGN),
                                                  tw_all + ((size_t)i << LOGN), pc, fpm.has(i), xcd_grouped_tile<TILE, A>(blockIdx.x, gridDim.x));
}

template <int A, int B, int TILE, typename Fp>
__global__ __launch_bounds__(TILE / kSmallE) void ntt_small_rows_moddown_kernel(
    Fp fpm, const uint64_t *conv, const TwPair *__restrict__ tw_all, const PrimeConst *__restrict__ pcs, const uint64_t *ip,
    uint64_t *out, const uint64_t *__restrict__ pinv, uint32_t nl, uint32_t K) {
    __shared__ uint64_t lds[(1 << B) * (TILE / (1 << B) + 1)];
    constexpr int LOGN = A + B;
    const uint32_t c = blockIdx.y & 1, i = blockIdx.y >> 1;
    const PrimeConst pc = pcs[i];
    const ModdownFoldEpi epi{ip + (((size_t)c * (nl + K) + i) << LOGN), out + (((size_t)c * nl + i) << LOGN),
                             pinv[2 * i], pinv[2 * i + 1], pc.q};
    ntt_rows_small_pe<A, B, true, TILE, kSmallE>(lds, BlkRawPro{conv + (((size_t)c * nl + i) << LOGN)},
                                                 tw_all + ((size_t)i << LOGN), pc, fpm.has(i), blockIdx.x, epi);
}

template <int A, int B, int TILE, bool KEEP_T, typename Fp>
__global__ __launch_bounds__(TILE / kSmallE) void ntt_small_cols_lift_kernel(
    Fp fpm, const uint64_t *last, uint64_t *lift, const TwPair *__restrict__ tw_all, const PrimeConst *__restrict__ pcs,
    const uint64_t *__restrict__ tab, uint32_t nl, uint32_t L) {
    __shared__ uint64_t lds[(1 << A) * (TILE / (1 << A) + 1)];
    constexpr int LOGN = A + B;
    const uint32_t l = nl - 1;
    const uint32_t c = blockIdx.y & 1, i = blockIdx.y >> 1;
    const PrimeConst pc = pcs[i];
    const LiftPro<KEEP_T> pro = lift_pro<KEEP_T, LOGN>(last, pcs, pc, tab, c, i, nl, L);
    ntt_cols_small_pro<A, B, true, TILE, kSmallE, true>(lds, pro, lift + (((size_t)c * l + i) << LOGN),
                                                  tw_all + ((size_t)i << LOGN), pc, fpm.has(i), xcd_grouped_tile<TILE, A>(blockIdx.x, gridDim.x));
}

template <int A, int B, int TILE, typename Fp>
__global__ __launch_bounds__(TILE / kSmallE) void ntt_small_rows_rescale_kernel(
    Fp fpm, const uint64_t *lift, const TwPair *__restrict__ tw_all, const PrimeConst *__restrict__ pcs, const uint64_t *in,
    uint64_t *out, const uint64_t *__restrict__ tab, uint32_t nl, uint32_t L) {
    __shared__ uint64_t lds[(1 << B) * (TILE / (1 << B) + 1)];
    constexpr int LOGN = A + B;
    const uint32_t l = nl - 1;
    const uint32_t c = blockIdx.y & 1, i = blockIdx.y >> 1;
    const PrimeConst pc = pcs[i];
    const uint64_t *t = tab + ((size_t)l * L + i) * 3;
    const RescaleTailEpi epi{in + (((size_t)c * nl + i) << LOGN), out + (((size_t)c * l + i) << LOGN), t[0], t[1],
                             pc.q};
    ntt_rows_small_pe<A, B, true, TILE, kSmallE>(lds, BlkRawPro{lift + (((size_t)c * l + i) << LOGN)},
                                                 tw_all + ((size_t)i << LOGN), pc, fpm.has(i), blockIdx.x, epi);
}

// First pass of INTT(d2) (galois == 0: d2 = a1 b1 of a, b) or of INTT(sigma_g(a1))
// on small tiles, into dc [nl][N].
template <int A, int B, int TILE, typename Fp>
__global__ __launch_bounds__(TILE / kSmallE) void ntt_small_inv_rows_first_kernel(
    Fp fpm, const uint64_t *a, const uint64_t *b, uint64_t *dc, uint32_t galois, const TwPair *__restrict__ tw_all,
    const PrimeConst *__restrict__ pcs, uint32_t nl) {
    __shared__ uint64_t lds[(1 << B) * (TILE / (1 << B) + 1)];
    constexpr int LOGN = A + B;
    const uint32_t i = blockIdx.y;
    const PrimeConst pc = pcs[i];
    const size_t li = (size_t)i << LOGN, poly = (size_t)nl << LOGN;
    if (galois) {
        const GatherPro pro{a + poly + li, galois, (uint32_t)LOGN};
        ntt_rows_small_pe<A, B, false, TILE, kSmallE>(lds, pro, tw_all + li, pc, fpm.has(i), blockIdx.x, BlkRawEpi{dc + li});
    } else {
        const TensorPro pro{a + poly + li, b + poly + li, pc.q, pc.r64, pc.r64_p, pc.one_p};
        ntt_rows_small_pe<A, B, false, TILE, kSmallE>(lds, pro, tw_all + li, pc, fpm.has(i), blockIdx.x, BlkRawEpi{dc + li});
    }
}


// Launchers: fpm is the context's FpMask, or NoFp where every limb of the launch is
// of a wide prime: a kernel that holds both forms is 0.3 to 0.5 us slower on those
// (N = 2^16, 8 limbs of 60 bits in a chain that ends in 45-bit ones: rescale 27.9
// against 27.2 us).
static bool narrow_in(const NttBatch &b) { return b.order.n_wide < b.per_poly; }
static bool narrow_in(const rf_ctx *c, uint32_t nl) { return c->q_order[nl].n_wide < nl; }

template <int A, int B, int TILE, int E, bool BLK, typename Fp>
static void launch_two_pass_small(const rf_ctx *c, Fp fpm, const NttBatch &b, bool forward, hipStream_t s,
                                  const PrimeConst *pcs) {
    const uint32_t limbs = b.per_poly * b.n_polys;
    const dim3 grid((1u << (A + B)) / TILE, limbs), block(TILE / E);
    NttBatch b2 = b;
    b2.in = b.out;
    b2.in_poly_stride = b.out_poly_stride;
    if (forward) {
        {
            ProfScope p("ntt_fwd_cols_small", s);
            hipLaunchKernelGGL((ntt_small_kernel<A, B, true, true, TILE, E, BLK>), grid, block, 0, s, b, fpm, c->d_tw_fwd, pcs);
        }
        ProfScope p("ntt_fwd_rows_small", s);
        hipLaunchKernelGGL((ntt_small_kernel<A, B, true, false, TILE, E, BLK>), grid, block, 0, s, b2, fpm, c->d_tw_fwd, pcs);
    } else {
        {
            ProfScope p("ntt_inv_rows_small", s);
            hipLaunchKernelGGL((ntt_small_kernel<A, B, false, false, TILE, E, BLK>), grid, block, 0, s, b, fpm, c->d_tw_inv,
                               pcs);
        }
        ProfScope p("ntt_inv_cols_small", s);
        hipLaunchKernelGGL((ntt_small_kernel<A, B, false, true, TILE, E, BLK>), grid, block, 0, s, b2, fpm, c->d_tw_inv, pcs);
    }
}

template <int A, int B, bool BLK, typename Fp>
static void launch_mixed(const rf_ctx *c, Fp fpm, const NttBatch &b, const MixGrid &m, dim3 grid, bool forward,
                         hipStream_t s, const PrimeConst *pcs) {
    const dim3 block(kThreads);
    NttBatch b2 = b;
    b2.in = b.out;
    b2.in_poly_stride = b.out_poly_stride;
    if (forward) {
        {
            ProfScope p("ntt_fwd_cols", s);
            hipLaunchKernelGGL((ntt_cols_kernel<A, B, true, BLK>), grid, block, 0, s, b, fpm, m, c->d_tw_fwd, pcs);
        }
        ProfScope p("ntt_fwd_rows", s);
        hipLaunchKernelGGL((ntt_rows_kernel<A, B, true, BLK>), grid, block, 0, s, b2, fpm, m, c->d_tw_fwd_rows, c->d_tw_fwd, pcs);
    } else {
        {
            ProfScope p("ntt_inv_rows", s);
            hipLaunchKernelGGL((ntt_rows_kernel<A, B, false, BLK>), grid, block, 0, s, b, fpm, m, c->d_tw_inv_rows, c->d_tw_inv,
                               pcs);
        }
        ProfScope p("ntt_inv_cols", s);
        hipLaunchKernelGGL((ntt_cols_kernel<A, B, false, BLK>), grid, block, 0, s, b2, fpm, m, c->d_tw_inv, pcs);
    }
}

template <int A, int B, bool BLK, typename Fp>
static void launch_two_pass_blk(const rf_ctx *c, Fp fpm, const NttBatch &b, bool forward, hipStream_t s,
                            const PrimeConst *pcs, const rf_tuning &tn) {
    const uint32_t limbs = b.per_poly * b.n_polys;
    const uint32_t tiles = limbs << (A + B - 12);
    if (tiles < tn.ntt_small_below) {
        const bool big = tn.ntt_small_tile == 2048 || (tn.ntt_small_tile == 0 && tiles * 2 >= tn.ntt_small_below);
        if (tn.ntt_small_radix == 8) {
            if (big) launch_two_pass_small<A, B, 2048, 8, BLK>(c, fpm, b, forward, s, pcs);
            else launch_two_pass_small<A, B, 1024, 8, BLK>(c, fpm, b, forward, s, pcs);
        } else {
            if (big) launch_two_pass_small<A, B, 2048, kSmallE, BLK>(c, fpm, b, forward, s, pcs);
            else launch_two_pass_small<A, B, 1024, kSmallE, BLK>(c, fpm, b, forward, s, pcs);
        }
        return;
    }
    MixGrid m{b.order, b.n_polys};
    if constexpr (!BLK) {
        if (m.o.n_wide == b.per_poly && tiles >= wide_tiles_from(c)) {
            // primes that follow each other need no look at the order, a load ahead of
            // all others (0.4 us of the passes at N = 2^13)
            if (!b.pmap) m.o = LimbOrder{nullptr, (uint16_t)b.per_poly, 0, (uint8_t)b.prime_base};
            launch_mixed<A, B, false>(c, WideTiles{}, b, m, dim3(tiles), forward, s, pcs);
            return;
        }
    }
    launch_mixed<A, B, BLK>(c, fpm, b, m, mix_grid(c, m.o.n_wide, b.per_poly, b.n_polys), forward, s, pcs);
}

template <int A, int B, typename Fp>
static void launch_two_pass(const rf_ctx *c, Fp fpm, const NttBatch &b, bool forward, hipStream_t s,
                            const PrimeConst *pcs, const rf_tuning &tn) {
    if (b.blocked) launch_two_pass_blk<A, B, true>(c, fpm, b, forward, s, pcs, tn);
    else launch_two_pass_blk<A, B, false>(c, fpm, b, forward, s, pcs, tn);
}

template <int A, int B, bool BLK, typename Fp>
static void launch_fwd_rows_blk(const rf_ctx *c, Fp fpm, const NttBatch &b, hipStream_t s, const rf_tuning &tn) {
    const uint32_t limbs = b.per_poly * b.n_polys;
    const uint32_t tiles = limbs << (A + B - 12);
    if (tiles < tn.ntt_small_below) {
        const bool big = tn.ntt_small_tile == 2048 || (tn.ntt_small_tile == 0 && tiles * 2 >= tn.ntt_small_below);
        ProfScope p("ntt_fwd_rows_small", s);
#define RF_FR(T, E)                                                                                              \
    hipLaunchKernelGGL((ntt_small_kernel<A, B, true, false, T, E, BLK>), dim3((1u << (A + B)) / T, limbs), dim3(T / E), 0, \
                       s, b, fpm, c->d_tw_fwd, c->d_pc)
        if (tn.ntt_small_radix == 8) {
            if (big) RF_FR(2048, 8);
            else RF_FR(1024, 8);
        } else {
            if (big) RF_FR(2048, kSmallE);
            else RF_FR(1024, kSmallE);
        }
#undef RF_FR
        return;
    }
    const MixGrid m{b.order, b.n_polys};
    ProfScope p("ntt_fwd_rows", s);
    hipLaunchKernelGGL((ntt_rows_kernel<A, B, true, BLK>), mix_grid(c, m.o.n_wide, b.per_poly, b.n_polys), dim3(kThreads), 0,
                       s, b, fpm, m, c->d_tw_fwd_rows, c->d_tw_fwd, c->d_pc);
}

template <int A, int B, typename Fp>
static void launch_fwd_rows(const rf_ctx *c, Fp fpm, const NttBatch &b, hipStream_t s, const rf_tuning &tn) {
    if (b.blocked) launch_fwd_rows_blk<A, B, true>(c, fpm, b, s, tn);
    else launch_fwd_rows_blk<A, B, false>(c, fpm, b, s, tn);
}

template <typename Fp>
static int launch_ntt_fwd_rows_t(const rf_ctx *c, Fp fpm, const NttBatch &b, hipStream_t s, const rf_tuning &tn) {
    if (b.per_poly * b.n_polys > 65535) return fail(RF_EUNSUPPORTED, "too many limbs in one NTT launch");
    switch (c->log_n) {
        case 13: launch_fwd_rows<7, 6>(c, fpm, b, s, tn); break;
        case 14: launch_fwd_rows<7, 7>(c, fpm, b, s, tn); break;
        case 15: launch_fwd_rows<8, 7>(c, fpm, b, s, tn); break;
        case 16: launch_fwd_rows<8, 8>(c, fpm, b, s, tn); break;
        default: return fail(RF_EUNSUPPORTED, "NTT row pass: ring degree");
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RF_EHIP, std::string("NTT launch: ") + hipGetErrorString(e));
    return RF_OK;
}

int launch_ntt_fwd_rows(const rf_ctx *c, const NttBatch &b, hipStream_t s, const rf_tuning *tn) {
    const rf_tuning &t = tn ? *tn : kDefaultTuning;
    return narrow_in(b) ? launch_ntt_fwd_rows_t(c, c->fp_mask, b, s, t) : launch_ntt_fwd_rows_t(c, NoFp{}, b, s, t);
}

// Small-tile size of a fused launch of `limbs` limbs, or 0 for the 4096-residue
// tiles (launch_two_pass's rule with the fused launches' threshold).
static int small_tile_of(const rf_ctx *c, uint32_t limbs, const rf_tuning *tn) {
    const rf_tuning &t = tn ? *tn : kDefaultTuning;
    const uint32_t tiles = limbs * (c->n / kTile);
    if (c->log_n < 13 || tiles >= t.ntt_fused_small_below) return 0;
    return t.ntt_small_tile == 2048 || (t.ntt_small_tile == 0 && tiles * 2 >= t.ntt_fused_small_below) ? 2048 : 1024;
}

template <typename Fp>
static int launch_ntt_fwd_moddown_t(const rf_ctx *c, Fp fpm, uint64_t *conv, const uint64_t *ip, uint64_t *out, uint32_t nl,
                           hipStream_t s, const rf_tuning *tn) {
    const uint64_t *tab = c->scheme == RF_BGV ? c->d_moddown_t : c->d_moddown;
    const uint64_t *cross = tab + moddown_cross_off(c), *negp = tab + moddown_negp_off(c);
    const uint64_t *pinv = c->d_moddown + moddown_pinv_off(c);
    const MixGrid mg = q_mix(c, nl, 2);
    const dim3 g = mix_grid(c, mg.o.n_wide, nl, 2);
    const int st = small_tile_of(c, 2 * nl, tn);
    // with narrow primes the conversion and the column pass are convert.hip's
    if constexpr (!std::is_same_v<Fp, NoFp>)
        if (const int rc = launch_moddown_cols(c, ip, conv, nl, s)) return rc;
    if (st) {
#define RF_SMDK(A, B, T, KP)                                                                                     \
    hipLaunchKernelGGL((ntt_small_cols_moddown_kernel<A, B, T, KP>), dim3(c->n / T, 2 * nl), dim3(T / kSmallE), 0, s, \
                       fpm, ip, conv, c->d_tw_fwd, c->d_pc, cross, negp, nl, c->L, c->K)
#define RF_SMD(A, B, T)                                                                                          \
    {                                                                                                            \
        if constexpr (std::is_same_v<Fp, NoFp>) {                                                                \
            ProfScope p("ntt_fwd_cols_moddown_small", s);                                                        \
            switch (c->K) {                                                                                      \
                case 1: RF_SMDK(A, B, T, 1); break;                                                              \
                case 2: RF_SMDK(A, B, T, 2); break;                                                              \
                case 3: RF_SMDK(A, B, T, 3); break;                                                              \
                case 4: RF_SMDK(A, B, T, 4); break;                                                              \
                default: RF_SMDK(A, B, T, 8); break;                                                             \
            }                                                                                                    \
        }                                                                                                        \
        ProfScope p("ntt_fwd_rows_moddown_small", s);                                                            \
        hipLaunchKernelGGL((ntt_small_rows_moddown_kernel<A, B, T>), dim3(c->n / T, 2 * nl), dim3(T / kSmallE), 0, s, \
                           fpm, conv, c->d_tw_fwd, c->d_pc, ip, out, pinv, nl, c->K);                            \
    }
#define RF_SMDT(A, B)                                                                                            \
    if (st == 2048) RF_SMD(A, B, 2048) else RF_SMD(A, B, 1024)
        switch (c->log_n) {
            case 13: RF_SMDT(7, 6) break;
            case 14: RF_SMDT(7, 7) break;
            case 15: RF_SMDT(8, 7) break;
            default: RF_SMDT(8, 8) break;
        }
#undef RF_SMDT
#undef RF_SMD
#undef RF_SMDK
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(RF_EHIP, std::string("NTT launch: ") + hipGetErrorString(e));
        return RF_OK;
    }
#define RF_MDK(A, B, KP)                                                                                         \
    hipLaunchKernelGGL((ntt_cols_moddown_kernel<A, B, KP>), g, dim3(kThreads),                                   \
                       0, s, fpm, mg, ip, conv, c->d_tw_fwd, c->d_pc, cross, negp, nl, c->L, c->K)
#define RF_MD(A, B)                                                                                              \
    {                                                                                                            \
        if constexpr (std::is_same_v<Fp, NoFp>) {                                                                \
            ProfScope p("ntt_fwd_cols_moddown", s);                                                              \
            switch (c->K) {                                                                                      \
                case 1: RF_MDK(A, B, 1); break;                                                                  \
                case 2: RF_MDK(A, B, 2); break;                                                                  \
                case 3: RF_MDK(A, B, 3); break;                                                                  \
                case 4: RF_MDK(A, B, 4); break;                                                                  \
                default: RF_MDK(A, B, 8); break;                                                                 \
            }                                                                                                    \
        }                                                                                                        \
        ProfScope p("ntt_fwd_rows_moddown", s);                                                                  \
        hipLaunchKernelGGL((ntt_rows_moddown_kernel<A, B>), g, dim3(kThreads), 0, s, fpm, mg, conv, c->d_tw_fwd_rows, c->d_tw_fwd, c->d_pc, ip, \
                           out, pinv, nl, c->K);                                                                 \
    }
    switch (c->log_n) {
        case 13: RF_MD(7, 6) break;
        case 14: RF_MD(7, 7) break;
        case 15: RF_MD(8, 7) break;
        case 16: RF_MD(8, 8) break;
        default: return fail(RF_EUNSUPPORTED, "fused ModDown NTT: ring degree");
    }
#undef RF_MD
#undef RF_MDK
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RF_EHIP, std::string("NTT launch: ") + hipGetErrorString(e));
    return RF_OK;
}

int launch_ntt_fwd_moddown(const rf_ctx *c, uint64_t *conv, const uint64_t *ip, uint64_t *out, uint32_t nl,
                           hipStream_t s, const rf_tuning *tn) {
    return narrow_in(c, nl) ? launch_ntt_fwd_moddown_t(c, c->fp_mask, conv, ip, out, nl, s, tn)
                            : launch_ntt_fwd_moddown_t(c, NoFp{}, conv, ip, out, nl, s, tn);
}

template <typename Fp>
static int launch_ntt_fwd_rescale_t(const rf_ctx *c, Fp fpm, const uint64_t *last, uint64_t *lift, const uint64_t *in,
                           uint64_t *out, uint32_t nl, bool keep_t, hipStream_t s, const rf_tuning *tn) {
    const uint32_t l = nl - 1;
    const MixGrid mg = q_mix(c, l, 2);
    const dim3 g = mix_grid(c, mg.o.n_wide, l, 2);
    const int st = small_tile_of(c, 2 * l, tn);
    const bool fused = lift_fused(c, nl);  // convert.hip has the INTT's last pass, the lift and the column pass
    if (fused)
        if (const int rc = launch_lift_cols(c, last, lift, nl, keep_t, s)) return rc;
    if (st) {
#define RF_SRS(A, B, T)                                                                                          \
    {                                                                                                            \
        const dim3 gs(c->n / T, 2 * l), bs(T / kSmallE);                                                         \
        if (!fused) {                                                                                            \
            ProfScope p("ntt_fwd_cols_lift_small", s);                                                           \
            if (keep_t)                                                                                          \
                hipLaunchKernelGGL((ntt_small_cols_lift_kernel<A, B, T, true>), gs, bs, 0, s, fpm, last, lift,   \
                                   c->d_tw_fwd, c->d_pc, c->d_rescale, nl, c->L);                                \
            else                                                                                                 \
                hipLaunchKernelGGL((ntt_small_cols_lift_kernel<A, B, T, false>), gs, bs, 0, s, fpm, last, lift,  \
                                   c->d_tw_fwd, c->d_pc, c->d_rescale, nl, c->L);                                \
        }                                                                                                        \
        ProfScope p("ntt_fwd_rows_rescale_small", s);                                                            \
        hipLaunchKernelGGL((ntt_small_rows_rescale_kernel<A, B, T>), gs, bs, 0, s, fpm, lift, c->d_tw_fwd, c->d_pc, in, \
                           out, c->d_rescale, nl, c->L);                                                         \
    }
#define RF_SRST(A, B)                                                                                            \
    if (st == 2048) RF_SRS(A, B, 2048) else RF_SRS(A, B, 1024)
        switch (c->log_n) {
            case 13: RF_SRST(7, 6) break;
            case 14: RF_SRST(7, 7) break;
            case 15: RF_SRST(8, 7) break;
            default: RF_SRST(8, 8) break;
        }
#undef RF_SRST
#undef RF_SRS
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(RF_EHIP, std::string("NTT launch: ") + hipGetErrorString(e));
        return RF_OK;
    }
#define RF_RS(A, B)                                                                                              \
    {                                                                                                            \
        if (!fused) {                                                                                            \
            ProfScope p("ntt_fwd_cols_lift", s);                                                                 \
            if (keep_t)                                                                                          \
                hipLaunchKernelGGL((ntt_cols_lift_kernel<A, B, true>), g, dim3(kThreads), 0, s, fpm, mg, last, lift, \
                                   c->d_tw_fwd, c->d_pc, c->d_rescale, nl, c->L);                                \
            else                                                                                                 \
                hipLaunchKernelGGL((ntt_cols_lift_kernel<A, B, false>), g, dim3(kThreads), 0, s, fpm, mg, last, lift, \
                                   c->d_tw_fwd, c->d_pc, c->d_rescale, nl, c->L);                                \
        }                                                                                                        \
        ProfScope p("ntt_fwd_rows_rescale", s);                                                                  \
        hipLaunchKernelGGL((ntt_rows_rescale_kernel<A, B>), g, dim3(kThreads), 0, s, fpm, mg, lift, c->d_tw_fwd_rows, c->d_tw_fwd, c->d_pc, in, \
                           out, c->d_rescale, nl, c->L);                                                         \
    }
    switch (c->log_n) {
        case 13: RF_RS(7, 6) break;
        case 14: RF_RS(7, 7) break;
        case 15: RF_RS(8, 7) break;
        case 16: RF_RS(8, 8) break;
        default: return fail(RF_EUNSUPPORTED, "fused rescale NTT: ring degree");
    }
#undef RF_RS
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RF_EHIP, std::string("NTT launch: ") + hipGetErrorString(e));
    return RF_OK;
}

int launch_ntt_fwd_rescale(const rf_ctx *c, const uint64_t *last, uint64_t *lift, const uint64_t *in,
                           uint64_t *out, uint32_t nl, bool keep_t, hipStream_t s, const rf_tuning *tn) {
    return narrow_in(c, nl - 1) ? launch_ntt_fwd_rescale_t(c, c->fp_mask, last, lift, in, out, nl, keep_t, s, tn)
                                : launch_ntt_fwd_rescale_t(c, NoFp{}, last, lift, in, out, nl, keep_t, s, tn);
}

template <typename Fp>
static int launch_intt_first_t(const rf_ctx *c, Fp fpm, const uint64_t *a, const uint64_t *b, uint64_t *dc, uint32_t galois,
                      uint32_t nl, hipStream_t s, const rf_tuning *tn) {
    const uint64_t N = c->n;
    const int st = small_tile_of(c, nl, tn);
    if (st) {
#define RF_SIF(A, B, T)                                                                                          \
    {                                                                                                            \
        const dim3 gs(c->n / T, nl), bs(T / kSmallE);                                                            \
        {                                                                                                        \
            ProfScope p(galois ? "ntt_inv_rows_gather_small" : "ntt_inv_rows_tensor_small", s);                  \
            hipLaunchKernelGGL((ntt_small_inv_rows_first_kernel<A, B, T>), gs, bs, 0, s, fpm, a, b, dc, galois,  \
                               c->d_tw_inv, c->d_pc, nl);                                                        \
        }                                                                                                        \
        NttBatch bc{dc, dc, 0, 0, nl, 1, 0, nullptr, {}};                                                        \
        ProfScope p("ntt_inv_cols_small", s);                                                                    \
        hipLaunchKernelGGL((ntt_small_kernel<A, B, false, true, T, kSmallE, true>), gs, bs, 0, s, bc, fpm, c->d_tw_inv, \
                           pc_modup(c, nl));                                                                     \
    }
#define RF_SIFT(A, B)                                                                                            \
    if (st == 2048) RF_SIF(A, B, 2048) else RF_SIF(A, B, 1024)
        switch (c->log_n) {
            case 13: RF_SIFT(7, 6) break;
            case 14: RF_SIFT(7, 7) break;
            case 15: RF_SIFT(8, 7) break;
            default: RF_SIFT(8, 8) break;
        }
#undef RF_SIFT
#undef RF_SIF
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(RF_EHIP, std::string("NTT launch: ") + hipGetErrorString(e));
        return RF_OK;
    }
#define RF_IF(A, B)                                                                                              \
    {                                                                                                            \
        const MixGrid mg = q_mix(c, nl, 1);                                                                      \
        const dim3 gr = mix_grid(c, mg.o.n_wide, nl, 1);                                                           \
        if (galois) {                                                                                            \
            ProfScope p("ntt_inv_rows_gather", s);                                                               \
            hipLaunchKernelGGL((ntt_inv_rows_gather_kernel<A, B>), gr, dim3(kThreads), 0, s, fpm, mg, a + (size_t)nl * N, dc, \
                               galois, c->d_tw_inv_rows, c->d_tw_inv, c->d_pc);                                  \
        } else {                                                                                                 \
            ProfScope p("ntt_inv_rows_tensor", s);                                                               \
            hipLaunchKernelGGL((ntt_inv_rows_tensor_kernel<A, B>), gr, dim3(kThreads), 0, s, fpm, mg, a, b, dc,  \
                               c->d_tw_inv_rows, c->d_tw_inv, c->d_pc, nl);                                      \
        }                                                                                                        \
        NttBatch bc{dc, dc, 0, 0, nl, 1, 0, nullptr, {}};                                                        \
        ProfScope p("ntt_inv_cols", s);                                                                          \
        hipLaunchKernelGGL((ntt_cols_kernel<A, B, false, true>), gr, dim3(kThreads), 0, s, bc, fpm, mg, c->d_tw_inv, pc_modup(c, nl)); \
    }
    switch (c->log_n) {
        case 13: RF_IF(7, 6) break;
        case 14: RF_IF(7, 7) break;
        case 15: RF_IF(8, 7) break;
        case 16: RF_IF(8, 8) break;
        default: return fail(RF_EUNSUPPORTED, "fused first INTT: ring degree");
    }
#undef RF_IF
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RF_EHIP, std::string("NTT launch: ") + hipGetErrorString(e));
    return RF_OK;
}

int launch_intt_first(const rf_ctx *c, const uint64_t *a, const uint64_t *b, uint64_t *dc, uint32_t galois,
                      uint32_t nl, hipStream_t s, const rf_tuning *tn) {
    return narrow_in(c, nl) ? launch_intt_first_t(c, c->fp_mask, a, b, dc, galois, nl, s, tn)
                            : launch_intt_first_t(c, NoFp{}, a, b, dc, galois, nl, s, tn);
}

template <typename Fp>
static int launch_ntt_t(const rf_ctx *c, Fp fpm, const NttBatch &b, bool forward, hipStream_t s, const PrimeConst *pcs,
               const rf_tuning *tn) {
    const uint32_t limbs = b.per_poly * b.n_polys;
    if (!pcs) pcs = c->d_pc;
    const rf_tuning &t = tn ? *tn : kDefaultTuning;
    if (limbs == 0) return RF_OK;
    if (limbs > 65535) return fail(RF_EUNSUPPORTED, "too many limbs in one NTT launch");
    switch (c->log_n) {
        case 12: return launch_ntt_single(c, b, forward, s, pcs);
        case 13: launch_two_pass<7, 6>(c, fpm, b, forward, s, pcs, t); break;
        case 14: launch_two_pass<7, 7>(c, fpm, b, forward, s, pcs, t); break;
        case 15: launch_two_pass<8, 7>(c, fpm, b, forward, s, pcs, t); break;
        case 16: launch_two_pass<8, 8>(c, fpm, b, forward, s, pcs, t); break;
        default: return fail(RF_EUNSUPPORTED, "ring degree");
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RF_EHIP, std::string("NTT launch: ") + hipGetErrorString(e));
    return RF_OK;
}

int launch_ntt(const rf_ctx *c, const NttBatch &b, bool forward, hipStream_t s, const PrimeConst *pcs,
               const rf_tuning *tn) {
    return narrow_in(b) ? launch_ntt_t(c, c->fp_mask, b, forward, s, pcs, tn)
                        : launch_ntt_t(c, NoFp{}, b, forward, s, pcs, tn);
}

template <int A, int B, typename Fp>
static void launch_inv_rows(const rf_ctx *c, Fp fpm, const NttBatch &b, hipStream_t s) {
    const uint32_t limbs = b.per_poly * b.n_polys;
    ProfScope p("ntt_inv_rows_small", s);
    hipLaunchKernelGGL((ntt_small_kernel<A, B, false, false, 1024, kSmallE, true>), dim3((1u << (A + B)) / 1024, limbs),
                       dim3(1024 / kSmallE), 0, s, b, fpm, c->d_tw_inv, c->d_pc);
}

template <typename Fp>
static int launch_intt_rows_t(const rf_ctx *c, Fp fpm, const NttBatch &b, hipStream_t s) {
    switch (c->log_n) {
        case 13: launch_inv_rows<7, 6>(c, fpm, b, s); break;
        case 14: launch_inv_rows<7, 7>(c, fpm, b, s); break;
        case 15: launch_inv_rows<8, 7>(c, fpm, b, s); break;
        case 16: launch_inv_rows<8, 8>(c, fpm, b, s); break;
        default: return fail(RF_EUNSUPPORTED, "INTT row pass: ring degree");
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RF_EHIP, std::string("NTT launch: ") + hipGetErrorString(e));
    return RF_OK;
}

int launch_intt_rows(const rf_ctx *c, const NttBatch &b, hipStream_t s) {
    return narrow_in(b) ? launch_intt_rows_t(c, c->fp_mask, b, s) : launch_intt_rows_t(c, NoFp{}, b, s);
}

template <int A, int B, bool BLK, typename Fp>
static void launch_inv_cols(const rf_ctx *c, Fp fpm, const NttBatch &b, hipStream_t s, const PrimeConst *pcs,
                            const rf_tuning &tn) {
    const uint32_t limbs = b.per_poly * b.n_polys;
    const uint32_t tiles = limbs << (A + B - 12);
    if (tiles < tn.ntt_small_below) {
        const bool big = tn.ntt_small_tile == 2048 || (tn.ntt_small_tile == 0 && tiles * 2 >= tn.ntt_small_below);
        ProfScope p("ntt_inv_cols_small", s);
#define RF_IC(T, E)                                                                                              \
    hipLaunchKernelGGL((ntt_small_kernel<A, B, false, true, T, E, BLK>), dim3((1u << (A + B)) / T, limbs), dim3(T / E), \
                       0, s, b, fpm, c->d_tw_inv, pcs)
        if (tn.ntt_small_radix == 8) {
            if (big) RF_IC(2048, 8);
            else RF_IC(1024, 8);
        } else {
            if (big) RF_IC(2048, kSmallE);
            else RF_IC(1024, kSmallE);
        }
#undef RF_IC
        return;
    }
    const MixGrid m{b.order, b.n_polys};
    ProfScope p("ntt_inv_cols", s);
    hipLaunchKernelGGL((ntt_cols_kernel<A, B, false, BLK>), mix_grid(c, m.o.n_wide, b.per_poly, b.n_polys),
                       dim3(kThreads), 0, s, b, fpm, m, c->d_tw_inv, pcs);
}

template <typename Fp>
static int launch_intt_cols_t(const rf_ctx *c, Fp fpm, const NttBatch &b, hipStream_t s, const PrimeConst *pcs,
                              const rf_tuning &tn) {
    if (b.per_poly * b.n_polys > 65535) return fail(RF_EUNSUPPORTED, "too many limbs in one NTT launch");
#define RF_IC(A, B)                                                                                              \
    if (b.blocked) launch_inv_cols<A, B, true>(c, fpm, b, s, pcs, tn);                                           \
    else launch_inv_cols<A, B, false>(c, fpm, b, s, pcs, tn)
    switch (c->log_n) {
        case 13: RF_IC(7, 6); break;
        case 14: RF_IC(7, 7); break;
        case 15: RF_IC(8, 7); break;
        case 16: RF_IC(8, 8); break;
        default: return fail(RF_EUNSUPPORTED, "INTT column pass: ring degree");
    }
#undef RF_IC
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RF_EHIP, std::string("NTT launch: ") + hipGetErrorString(e));
    return RF_OK;
}

int launch_intt_cols(const rf_ctx *c, const NttBatch &b, hipStream_t s, const PrimeConst *pcs, const rf_tuning *tn,
                     bool mixed) {
    const rf_tuning &t = tn ? *tn : kDefaultTuning;
    if (!pcs) pcs = c->d_pc;
    return mixed || narrow_in(b) ? launch_intt_cols_t(c, c->fp_mask, b, s, pcs, t)
                        : launch_intt_cols_t(c, NoFp{}, b, s, pcs, t);
}

}  // namespace rf
