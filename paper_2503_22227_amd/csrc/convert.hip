// Base conversions inside the first pass of the NTT that follows them: ModUp
// (the digits' extension) and ModDown; the device code is in conv_dev.hpp.
#include <hip/hip_runtime.h>

#include "conv_dev.hpp"

namespace rf {

struct ConvArgs {
    const ConvUnit *units;
    const TwPair *tw;
    const PrimeConst *pcs;
    const int8_t *frag;
    const double *off;
    uint32_t nl, L, K, alpha;
};

// grid.x: units x tiles of 1024 residues; the wide units come first, since their
// integer arithmetic takes longest.
// BLK false: natural layouts (coefficients given by the caller: BFV, digits of one limb).
template <int A, int B, int KP, bool BLK, typename Fp>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void modup_cols_kernel(
    ConvArgs c, const uint64_t *x, uint64_t *ext, const uint64_t *__restrict__ tab, size_t tab_stride) {
    __shared__ uint64_t lds[conv_lds<A, Fp>()];
    constexpr int LOGN = A + B, TL = LOGN - 10;
    const int tile = xcd_grouped_tile<kMixTile, A>(blockIdx.x & ((1 << TL) - 1), 1 << TL);
    const ConvUnit *un = c.units + (blockIdx.x >> TL);
    const uint32_t j = un->digit, s = un->size, blk = j * c.alpha + s - 1;
    const uint64_t *src = x + ((size_t)j * c.alpha << LOGN);
    uint64_t *dst = ext + ((size_t)j * (c.nl + c.K - c.alpha) << LOGN);
    if (std::is_same_v<Fp, NoFp> || un->wide) {
        const uint32_t li = un->e[0] & 0xffffu, g = un->e[0] >> 16;
        const PrimeConst pc = c.pcs[g];
        const ModupColsPro<KP> pro =
            modup_cols_pro<KP, LOGN>(src, s, tab + blk * tab_stride + 2 * c.alpha + (size_t)g * c.alpha, pc);
        ntt_cols_small_t<ArInt, A, B, true, kMixTile, kMixE, BLK>(lds, pro, dst + ((size_t)li << LOGN),
                                                             c.tw + ((size_t)g << LOGN), ArInt(pc), tile);
    } else if constexpr (!std::is_same_v<Fp, NoFp>) {
        constexpr int KB = KP <= 4 ? 4 : 8;
        const size_t b = (size_t)blk * (c.L + c.K);
        conv_cols_narrow<A, B, KB, false, BLK>(lds, src, s, nullptr, c.frag + b * (64 * KB), c.off + b, c.tw, c.pcs, un, dst,
                                          tile);
    }
}

template <int A, int B, int KP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void moddown_cols_kernel(
    ConvArgs c, const uint64_t *ip, uint64_t *conv, const uint64_t *__restrict__ cross,
    const uint64_t *__restrict__ negp) {
    __shared__ uint64_t lds[conv_lds<A, FpMask>()];
    constexpr int LOGN = A + B, TL = LOGN - 10;
    const int tile = xcd_grouped_tile<kMixTile, A>(blockIdx.x & ((1 << TL) - 1), 1 << TL);
    const uint32_t u = blockIdx.x >> TL, poly = u & 1;
    const ConvUnit *un = c.units + (u >> 1);
    uint64_t *dst = conv + ((size_t)poly * c.nl << LOGN);
    if (un->wide) {
        const uint32_t i = un->e[0] & 0xffffu;
        const PrimeConst pc = c.pcs[i];
        const ModdownPro<KP> pro = moddown_pro<KP, LOGN>(ip, c.pcs, pc, cross, negp, poly, i, c.nl, c.L, c.K);
        ntt_cols_small_t<ArInt, A, B, true, kMixTile, kMixE, true>(lds, pro, dst + ((size_t)i << LOGN),
                                                             c.tw + ((size_t)i << LOGN), ArInt(pc), tile);
    } else {
        constexpr int KB = KP <= 4 ? 4 : 8;
        conv_cols_narrow<A, B, KB, true, true>(lds, ip + (((size_t)poly * (c.nl + c.K) + c.nl) << LOGN), c.K, c.pcs + c.L,
                                         c.frag, c.off, c.tw, c.pcs, un, dst, tile);
    }
}

// Last pass of the INTT of the dropped limb (last [2][N] after its row pass), the
// lift and the column pass of its targets, units as moddown's: every workgroup
// transforms the tile of the dropped limb for itself, for up to four targets.  The
// INTT's pass had a launch of 128 workgroups: with it N = 2^16, 46 targets 17.5 us
// against 7.0 + 14.2, N = 2^14, 20 targets 9.4 against 4.5 + 5.0 and a launch less
// for the host.  Bound by latency; the targets' twiddles fetched before the
// dropped limb's pass spill (19.1).
template <int A, int B, bool KEEP_T>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void lift_cols_kernel(
    ConvArgs c, FpMask fpm, const uint64_t *last, uint64_t *lift, const TwPair *__restrict__ tw_inv,
    const uint64_t *__restrict__ tab) {
    __shared__ uint64_t lds[conv_lds<A, FpMask>()];
    constexpr int LOGN = A + B, TL = LOGN - 10;
    const int tile = xcd_grouped_tile<kMixTile, A>(blockIdx.x & ((1 << TL) - 1), 1 << TL);
    const uint32_t u = blockIdx.x >> TL, poly = u & 1, l = c.nl - 1;
    const ConvUnit *un = c.units + (u >> 1);
    const PrimeConst pl = c.pcs[l];
    const TwPair *tw = tw_inv + ((size_t)l << LOGN);
    if (fpm.has(l)) inv_cols_lds<ArFp, A, B>(lds, last + ((size_t)poly << LOGN), tw, ArFp(pl), tile);
    else inv_cols_lds<ArInt, A, B>(lds, last + ((size_t)poly << LOGN), tw, ArInt(pl), tile);
    uint64_t *dst = lift + ((size_t)poly * l << LOGN);
    if (un->wide) lift_cols_wide<A, B, KEEP_T>(lds, c.pcs, tab, c.tw, un->e[0] & 0xffffu, dst, c.nl, c.L, tile);
    else lift_cols_narrow<A, B, KEEP_T>(lds, c.pcs, tab, c.tw, un, dst, c.nl, c.L, tile);
}

static int check_conv() {
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? RF_OK : fail(RF_EHIP, std::string("conversion launch: ") + hipGetErrorString(e));
}

// Wide targets convert on integer units, a workgroup each: with digits of one limb
// that is one product (the separate conversion took 8 us of 112 of a product and
// modulus switch at N = 2^15, 9 + 1 limbs), with more it would read every source
// again for each target (64.6 us for what two launches do in 43.3, 56 targets
// from 8 sources at N = 2^16), so bases of wide primes alone keep two launches.
// A single source needs no input factor: Q_j / q_i = 1.
bool modup_fused(const rf_ctx *c, bool scaled) {
    return c->log_n >= 13 && (c->alpha == 1 || (scaled && c->fp_mask.any()));
}

template <int A, int B>
static void modup_cols(const rf_ctx *c, const ConvArgs &a, dim3 grid, const uint64_t *x, uint64_t *ext,
                       bool blocked, hipStream_t s) {
#define RF_MU(KP, BLK, FP)                                                                                       \
    hipLaunchKernelGGL((modup_cols_kernel<A, B, KP, BLK, FP>), grid, dim3(kThreads), 0, s, a, x, ext, c->d_modup, c->modup_stride)
    const bool fp = c->fp_mask.any();
    if (c->alpha == 1) {
        if (blocked) {
            if (fp) RF_MU(1, true, FpMask);
            else RF_MU(1, true, NoFp);
        } else {
            if (fp) RF_MU(1, false, FpMask);
            else RF_MU(1, false, NoFp);
        }
    } else if (c->alpha <= 4) {
        RF_MU(4, true, FpMask);
    } else {
        RF_MU(8, true, FpMask);
    }
#undef RF_MU
}

int launch_modup_cols(const rf_ctx *c, const uint64_t *x, uint64_t *ext, uint32_t nl, bool blocked, hipStream_t s) {
    const rf_ctx::UnitRef u = c->modup_units[nl];
    const ConvArgs a{c->d_units + u.off, c->d_tw_fwd, c->d_pc, c->d_conv_mu, c->d_conv_mu_off, nl, c->L, c->K, c->alpha};
    const dim3 grid(u.n * (c->n / kMixTile));
    ProfScope p("modup_cols", s);
    switch (c->log_n) {
        case 13: modup_cols<7, 6>(c, a, grid, x, ext, blocked, s); break;
        case 14: modup_cols<7, 7>(c, a, grid, x, ext, blocked, s); break;
        case 15: modup_cols<8, 7>(c, a, grid, x, ext, blocked, s); break;
        case 16: modup_cols<8, 8>(c, a, grid, x, ext, blocked, s); break;
        default: return fail(RF_EUNSUPPORTED, "ModUp column pass: ring degree");
    }
    return check_conv();
}

template <int A, int B>
static void moddown_cols(const rf_ctx *c, const ConvArgs &a, dim3 grid, const uint64_t *ip, uint64_t *conv,
                         const uint64_t *cross, const uint64_t *negp, hipStream_t s) {
#define RF_MD(KP) hipLaunchKernelGGL((moddown_cols_kernel<A, B, KP>), grid, dim3(kThreads), 0, s, a, ip, conv, cross, negp)
    switch (c->K) {
        case 1: RF_MD(1); break;
        case 2: RF_MD(2); break;
        case 3: RF_MD(3); break;
        case 4: RF_MD(4); break;
        default: RF_MD(8); break;
    }
#undef RF_MD
}

int launch_moddown_cols(const rf_ctx *c, const uint64_t *ip, uint64_t *conv, uint32_t nl, hipStream_t s) {
    const rf_ctx::UnitRef u = c->moddown_units[nl];
    const ConvArgs a{c->d_units + u.off, c->d_tw_fwd, c->d_pc, c->d_conv_md, c->d_conv_md_off, nl, c->L, c->K, c->alpha};
    const uint64_t *tab = c->scheme == RF_BGV ? c->d_moddown_t : c->d_moddown;
    const uint64_t *cross = tab + moddown_cross_off(c), *negp = tab + moddown_negp_off(c);
    const dim3 grid(2 * u.n * (c->n / kMixTile));
    ProfScope p("moddown_cols", s);
    switch (c->log_n) {
        case 13: moddown_cols<7, 6>(c, a, grid, ip, conv, cross, negp, s); break;
        case 14: moddown_cols<7, 7>(c, a, grid, ip, conv, cross, negp, s); break;
        case 15: moddown_cols<8, 7>(c, a, grid, ip, conv, cross, negp, s); break;
        case 16: moddown_cols<8, 8>(c, a, grid, ip, conv, cross, negp, s); break;
        default: return fail(RF_EUNSUPPORTED, "ModDown column pass: ring degree");
    }
    return check_conv();
}

template <int A, int B>
static void lift_cols(const rf_ctx *c, const ConvArgs &a, dim3 grid, const uint64_t *last, uint64_t *lift, bool keep_t,
                      hipStream_t s) {
    if (keep_t)
        hipLaunchKernelGGL((lift_cols_kernel<A, B, true>), grid, dim3(kThreads), 0, s, a, c->fp_mask, last, lift,
                           c->d_tw_inv, c->d_rescale);
    else
        hipLaunchKernelGGL((lift_cols_kernel<A, B, false>), grid, dim3(kThreads), 0, s, a, c->fp_mask, last, lift,
                           c->d_tw_inv, c->d_rescale);
}

// A wide target's workgroup transforms the dropped limb's tile for itself alone: with
// 10 wide targets of 19 a rescale at N = 2^16 takes 41.6 us against 43.2, with 16 of
// 19 44.5 against 42.5.
bool lift_fused(const rf_ctx *c, uint32_t nl) {
    return c->fp_mask.any() && 4 * c->q_order[nl - 1].n_wide <= 3 * (nl - 1);
}

int launch_lift_cols(const rf_ctx *c, const uint64_t *last, uint64_t *lift, uint32_t nl, bool keep_t, hipStream_t s) {
    const rf_ctx::UnitRef u = c->moddown_units[nl - 1];
    const ConvArgs a{c->d_units + u.off, c->d_tw_fwd, c->d_pc, nullptr, nullptr, nl, c->L, c->K, c->alpha};
    const dim3 grid(2 * u.n * (c->n / kMixTile));
    ProfScope p("lift_cols", s);
    switch (c->log_n) {
        case 13: lift_cols<7, 6>(c, a, grid, last, lift, keep_t, s); break;
        case 14: lift_cols<7, 7>(c, a, grid, last, lift, keep_t, s); break;
        case 15: lift_cols<8, 7>(c, a, grid, last, lift, keep_t, s); break;
        case 16: lift_cols<8, 8>(c, a, grid, last, lift, keep_t, s); break;
        default: return fail(RF_EUNSUPPORTED, "lift column pass: ring degree");
    }
    return check_conv();
}

}  // namespace rf
